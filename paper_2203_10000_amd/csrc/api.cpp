// C-ABI entry points: contexts, surface sets, point labeling.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>

#include "runtime.h"

namespace sal {

static thread_local std::string g_last_error;

sal_status set_error(sal_status s, const std::string &msg) {
    g_last_error = msg;
    return s;
}

sal_status hip_error(hipError_t e, const char *what) {
    g_last_error = std::string(what) + ": " + hipGetErrorString(e);
    return e == hipErrorOutOfMemory ? SAL_ERR_OUT_OF_MEMORY : SAL_ERR_DEVICE;
}

namespace {

// Replaces *p by a buffer of n entries; the old one must be out of use.
template <typename T>
sal_status renew(T **p, int64_t n) {
    if (*p) (void)hipFree(*p);
    *p = nullptr;
    SAL_HIP(dev_malloc((void **)p, (size_t)n * sizeof(T)));
    return SAL_OK;
}

}  // namespace

sal_status ensure_label_scratch(sal_context *ctx, const ScratchSize &need) {
    sal_status st;
    if (need.points > ctx->point_cap || need.tiles > ctx->tile_cap || need.insts > ctx->inst_cap ||
        need.spans > ctx->span_cap || need.pairs > ctx->pair_cap) {
        SAL_HIP(hipStreamSynchronize(ctx->stream));
        ctx->batch_graph_fields.clear();   // a captured batch graph points at the old buffers
    }
    if (need.points > ctx->point_cap) {
        ctx->point_cap = 0;
        if ((st = renew(&ctx->flag_list, need.points)) != SAL_OK ||
            (st = renew(&ctx->ord_idx1, need.points)) != SAL_OK ||
            (st = renew(&ctx->ord_key1, need.points)) != SAL_OK ||
            (st = renew(&ctx->ord_perm, need.points)) != SAL_OK)
            return st;
        ctx->point_cap = need.points;
    }
    if (need.tiles > ctx->tile_cap) {
        ctx->tile_cap = 0;
        if ((st = renew(&ctx->ord_hist, need.tiles * kOrderBins)) != SAL_OK) return st;
        ctx->tile_cap = need.tiles;
    }
    if (need.insts > ctx->inst_cap) {
        ctx->inst_cap = 0;
        if ((st = renew(&ctx->ord_tot, need.insts * kOrderBins)) != SAL_OK) return st;
        ctx->inst_cap = need.insts;
    }
    if (need.spans > ctx->span_cap) {
        ctx->span_cap = 0;
        if ((st = renew(&ctx->span_w, need.spans)) != SAL_OK || (st = renew(&ctx->open_spans, need.spans)) != SAL_OK)
            return st;
        ctx->span_cap = need.spans;
    }
    if (need.pairs > ctx->pair_cap) {
        ctx->pair_cap = 0;
        if ((st = renew(&ctx->pairs, need.pairs)) != SAL_OK) return st;
        ctx->pair_cap = need.pairs;
    }
    return SAL_OK;
}

sal_status ensure_label_scratch(sal_context *ctx, const sal_surface_set *set, int64_t n) {
    return ensure_label_scratch(ctx, label_scratch_size(n, set->n_surf));
}

sal_status resolve_options(const sal_label_options *in, sal_label_options *out) {
    sal_label_options_default(out);
    if (in) *out = *in;
    if (out->precision != SAL_PREC_FP64 && out->precision != SAL_PREC_FP32_RECHECK)
        return set_error(SAL_ERR_INVALID_ARG, "precision must be SAL_PREC_FP64 or SAL_PREC_FP32_RECHECK");
    if (out->winding_type < SAL_WINDING_NONE || out->winding_type > SAL_WINDING_F64)
        return set_error(SAL_ERR_INVALID_ARG, "bad winding_type");
    if (!(out->threshold > 0.0 && out->threshold < 1.0))
        return set_error(SAL_ERR_INVALID_ARG, "threshold must be in (0, 1)");
    if (!(out->recheck_band >= 0.0 && out->recheck_band < 1.0))
        return set_error(SAL_ERR_INVALID_ARG, "recheck_band must be in [0, 1)");
    if (out->kappa == 0.0) out->kappa = 0.03125;
    if (!(out->kappa > 0.0 && out->kappa < 1.0))
        return set_error(SAL_ERR_INVALID_ARG, "kappa must be in (0, 1)");
    if (out->points_per_lane != 0 && out->points_per_lane != 1 && out->points_per_lane != 2 &&
        out->points_per_lane != 4)
        return set_error(SAL_ERR_INVALID_ARG, "points_per_lane must be 0, 1, 2 or 4");
    if (out->block_waves != 0 && out->block_waves != 1 && out->block_waves != 2 && out->block_waves != 4 &&
        out->block_waves != 8)
        return set_error(SAL_ERR_INVALID_ARG, "block_waves must be 0, 1, 2, 4 or 8");
    if (out->element_rule != SAL_RULE_CENTROID && out->element_rule != SAL_RULE_FOUR_NODES)
        return set_error(SAL_ERR_INVALID_ARG, "element_rule must be SAL_RULE_CENTROID or SAL_RULE_FOUR_NODES");
    return SAL_OK;
}

LabelScratch context_scratch(const sal_context *ctx) {
    return LabelScratch{ctx->counters, ctx->flag_list, ctx->work, ctx->span_w, ctx->open_spans, ctx->pairs,
                        OrderScratch{ctx->ord_idx1, ctx->ord_key1, ctx->ord_perm, ctx->ord_hist, ctx->ord_tot}};
}

LabelInst make_inst(const sal_surface_set *set, int64_t n, const float *x, const float *y, const float *z,
                    int32_t *labels, void *winding, int64_t wstride, unsigned long long *masks,
                    unsigned long long *counters) {
    LabelInst in{};
    in.rec = set->rec;
    in.surf = set->surf;
    in.ent = set->ent;
    in.leaf = set->leaf;
    in.x = x;
    in.y = y;
    in.z = z;
    in.labels = labels;
    in.winding = winding;
    in.masks = masks;
    in.counters = counters;
    in.n = n;
    in.wstride = wstride;
    in.n_surf = set->n_surf;
    in.tile = order_tile(n);
    in.n_tiles = (int32_t)order_tiles(n);
    for (int c = 0; c < 3; ++c) {
        in.lo[c] = set->lo[c];
        in.scale[c] = 128.0f / (set->hi[c] - set->lo[c]);
    }
    return in;
}

sal_status enqueue_label_on(sal_context *ctx, const sal_surface_set *set, int64_t n,
                            const int64_t *n_dev, const float *x, const float *y, const float *z,
                            const sal_label_options &opt, int32_t *labels, void *winding,
                            hipEvent_t ev_mid, hipStream_t stream, unsigned long long *masks) {
    return enqueue_label_with(ctx, set, n, n_dev, x, y, z, opt, labels, winding, ev_mid, stream,
                              masks, context_scratch(ctx));
}

sal_status enqueue_label_with(sal_context *ctx, const sal_surface_set *set, int64_t n,
                              const int64_t *n_dev, const float *x, const float *y,
                              const float *z, const sal_label_options &opt, int32_t *labels,
                              void *winding, hipEvent_t ev_mid, hipStream_t stream,
                              unsigned long long *masks, const LabelScratch &sc) {
    const bool fp64 = opt.precision == SAL_PREC_FP64;
    LabelArgs a{};
    a.winding_type = winding ? opt.winding_type : SAL_WINDING_NONE;
    a.n_dev = n_dev;
    a.threshold = opt.threshold;
    a.band = opt.recheck_band;
    a.kappa = (float)opt.kappa;
    a.cull = opt.cull_bounds ? 1 : 0;
    a.flag_list = sc.flag_list;
    a.work = sc.work;
    a.open_spans = sc.open_spans;
    a.pairs = sc.pairs;
    a.ord = sc.ord;
    const size_t wsize = opt.winding_type == SAL_WINDING_F64 ? sizeof(double) : sizeof(float);
    for (int64_t at = 0; at < n; at += kChunkPoints) {
        const int64_t m = n - at < kChunkPoints ? n - at : kChunkPoints;
        a.n_dev_skip = at;
        a.one = make_inst(set, m, x + at, y + at, z + at, labels + at,
                          winding ? (char *)winding + (size_t)at * wsize : nullptr, n,
                          masks ? masks + at : nullptr, sc.counters);
        if (n <= kPointFormMax) {
            // so few points that a wavefront each leaves the chip half empty:
            // the surfaces are shared out too
            const bool spread = set->n_surf > 1 && opt.block_waves > 1 && m <= (int64_t)ctx->n_cu * 8;
            SAL_HIP(launch_label_point(a, fp64, spread, m, opt.block_waves, stream));
            continue;
        }
        SAL_HIP(launch_order(a, a.one.n_tiles, stream));
        a.span_w = m * set->n_surf >= kSpanPairs ? sc.span_w : nullptr;
        a.n_pairs = group_count(m) * set->n_surf;
        if (a.span_w) SAL_HIP(launch_label_span(a, span_count(m) * set->n_surf, stream));
        SAL_HIP(launch_label_pair(a, fp64, std::min<int64_t>(a.n_pairs, (int64_t)ctx->n_cu * kPairWaves),
                                  opt.block_waves, stream));
        SAL_HIP(launch_label_final(a, fp64, group_count(m), stream));
        if (ev_mid && at + m == n) SAL_HIP(hipEventRecord(ev_mid, stream));
        SAL_HIP(launch_recheck(a, fp64, ctx->n_cu * 8, stream));
    }
    if (ev_mid && n <= kPointFormMax) SAL_HIP(hipEventRecord(ev_mid, stream));
    return SAL_OK;
}

sal_status enqueue_label(sal_context *ctx, const sal_surface_set *set, int64_t n, const float *x,
                         const float *y, const float *z, const sal_label_options &opt_in,
                         int32_t *labels, void *winding, hipEvent_t ev_start, hipEvent_t ev_mid,
                         int *shape, unsigned long long *masks) {
    sal_label_options opt = opt_in;
    sal_status ts = tune_launch(ctx, set, n, x, y, z, labels, &opt);
    if (ts != SAL_OK) return ts;
    if (ev_start) SAL_HIP(hipEventRecord(ev_start, ctx->stream));
    if (shape) {
        shape[0] = opt.points_per_lane;
        shape[1] = opt.block_waves;
    }
    return enqueue_label_on(ctx, set, n, nullptr, x, y, z, opt, labels, winding, ev_mid,
                            ctx->stream, masks);
}

}  // namespace sal

using namespace sal;

#define SAL_GUARD_BEGIN try {
#define SAL_GUARD_END                                                          \
    }                                                                          \
    catch (const std::bad_alloc &) {                                           \
        return set_error(SAL_ERR_OUT_OF_MEMORY, "host allocation failed");     \
    }                                                                          \
    catch (const std::exception &ex) {                                         \
        return set_error(SAL_ERR_INTERNAL, ex.what());                         \
    }                                                                          \
    catch (...) {                                                              \
        return set_error(SAL_ERR_INTERNAL, "unknown exception");               \
    }

extern "C" {

const char *sal_status_string(sal_status s) {
    switch (s) {
        case SAL_OK: return "ok";
        case SAL_ERR_INVALID_ARG: return "invalid argument";
        case SAL_ERR_NOT_CLOSED: return "surface not closed";
        case SAL_ERR_ORIENTATION: return "surface orientation";
        case SAL_ERR_OUT_OF_MEMORY: return "out of memory";
        case SAL_ERR_DEVICE: return "device error";
        case SAL_ERR_CAPACITY: return "capacity exceeded";
        case SAL_ERR_INTERNAL: return "internal error";
    }
    return "unknown status";
}

const char *sal_last_error_message(void) { return g_last_error.c_str(); }

int sal_abi_version(void) { return SAL_ABI_VERSION; }

void sal_debug_fail_allocation(int64_t n) { sal::fail_allocation(n); }

void sal_label_options_default(sal_label_options *o) {
    if (!o) return;
    std::memset(o, 0, sizeof(*o));
    o->precision = SAL_PREC_FP32_RECHECK;
    o->winding_type = SAL_WINDING_NONE;
    o->threshold = 0.5;
    o->recheck_band = 1e-3;
    o->kappa = 0.0;
    o->points_per_lane = 0;
    o->block_waves = 0;
    o->use_graph = 0;
    o->element_rule = SAL_RULE_CENTROID;
}

sal_status sal_context_create(int device, void *stream, sal_context **out) {
    SAL_GUARD_BEGIN
    g_last_error.clear();
    if (!out) return set_error(SAL_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    int count = 0;
    hipError_t e = hipGetDeviceCount(&count);
    if (e != hipSuccess || count == 0) return set_error(SAL_ERR_DEVICE, "no HIP device available");
    if (device < 0 || device >= count) return set_error(SAL_ERR_INVALID_ARG, "device out of range");
    SAL_HIP(hipSetDevice(device));
    auto *ctx = new sal_context();
    ctx->device = device;
    pool_add_context();
    ctx->stream = (hipStream_t)stream;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) == hipSuccess) ctx->n_cu = prop.multiProcessorCount;
    if (ctx->n_cu <= 0) ctx->n_cu = 256;
    // set-up of sal_label_points_noalloc: its scratch array's address on
    // this device (looked up once per device; a failure shows there)
    (void)noalloc_scratch(device);
    for (auto &ev : ctx->ev) {
        e = hipEventCreate(&ev);
        if (e != hipSuccess) { sal_context_destroy(ctx); return hip_error(e, "hipEventCreate"); }
    }
    e = dev_malloc((void **)&ctx->counters, kNumCounters * sizeof(unsigned long long));
    if (e != hipSuccess) { sal_context_destroy(ctx); return hip_error(e, "hipMalloc(counters)"); }
    e = dev_malloc((void **)&ctx->tune_counters, kNumCounters * sizeof(unsigned long long));
    if (e != hipSuccess) { sal_context_destroy(ctx); return hip_error(e, "hipMalloc(counters)"); }
    e = dev_malloc((void **)&ctx->work, kNumWork * sizeof(unsigned long long));
    if (e != hipSuccess) { sal_context_destroy(ctx); return hip_error(e, "hipMalloc(work counters)"); }
    e = hipHostMalloc((void **)&ctx->host_words, 16 * sizeof(int64_t), hipHostMallocDefault);
    if (e != hipSuccess) { sal_context_destroy(ctx); return hip_error(e, "hipHostMalloc(host words)"); }
    e = hipStreamCreateWithFlags(&ctx->capture_stream, hipStreamNonBlocking);
    if (e != hipSuccess) { sal_context_destroy(ctx); return hip_error(e, "hipStreamCreate"); }
    *out = ctx;
    return SAL_OK;
    SAL_GUARD_END
}

sal_status sal_context_set_stream(sal_context *ctx, void *stream) {
    if (!ctx) return set_error(SAL_ERR_INVALID_ARG, "ctx is NULL");
    ctx->stream = (hipStream_t)stream;
    ctx->stream_token = new_stream_token();
    return SAL_OK;
}

void sal_context_destroy(sal_context *ctx) {
    if (!ctx) return;
    (void)hipSetDevice(ctx->device);
    const bool idle = hipStreamSynchronize(ctx->stream) == hipSuccess;
    for (auto &ev : ctx->ev)
        if (ev) (void)hipEventDestroy(ev);
    if (ctx->batch_graph) (void)hipGraphExecDestroy(ctx->batch_graph);
    void *bufs[] = {ctx->flag_list, ctx->ord_idx1, ctx->ord_key1,    ctx->ord_perm,      ctx->ord_hist,
                    ctx->ord_tot,   ctx->work,     ctx->span_w,      ctx->open_spans, ctx->pairs,
                    ctx->counters,    ctx->tune_counters, ctx->batch_insts,
                    ctx->batch_counters};
    for (void *p : bufs)
        if (p) (void)hipFree(p);
    if (ctx->host_words) (void)hipHostFree(ctx->host_words);
    if (ctx->capture_stream) (void)hipStreamDestroy(ctx->capture_stream);
    pool_remove_context(idle ? ctx->stream_token : 0);
    delete ctx;
}

sal_status sal_surface_set_create(sal_context *ctx, const sal_surface_desc *s, int32_t n,
                                  uint32_t flags, sal_surface_set **out) {
    SAL_GUARD_BEGIN
    g_last_error.clear();
    if (out) *out = nullptr;
    if (flags & ~SAL_SURF_AUTO_ORIENT) return set_error(SAL_ERR_INVALID_ARG, "unknown flag bits");
    return build_surface_set(ctx, s, n, flags, out);
    SAL_GUARD_END
}

void sal_surface_set_destroy(sal_surface_set *set) { destroy_surface_set(set); }

sal_status sal_surface_set_get_info(const sal_surface_set *set, sal_surface_set_info *info) {
    if (!set || !info) return set_error(SAL_ERR_INVALID_ARG, "NULL argument");
    info->n_surfaces = set->n_surf;
    info->n_triangles = set->n_tri;
    info->n_strips = set->n_strips;
    info->device_bytes = set->bytes;
    return SAL_OK;
}

sal_status sal_label_points(sal_context *ctx, const sal_surface_set *set, int64_t n,
                            const float *x, const float *y, const float *z,
                            const sal_label_options *opt_in, int32_t *labels, void *winding,
                            sal_label_stats *stats) {
    SAL_GUARD_BEGIN
    g_last_error.clear();
    if (!ctx || !set) return set_error(SAL_ERR_INVALID_ARG, "ctx or set is NULL");
    if (n < 0) return set_error(SAL_ERR_INVALID_ARG, "n_points < 0");
    if (set->device != ctx->device)
        return set_error(SAL_ERR_INVALID_ARG, "surface set lives on another device");
    sal_label_options opt;
    sal_status st = resolve_options(opt_in, &opt);
    if (st != SAL_OK) return st;
    if (winding && opt.winding_type == SAL_WINDING_NONE)
        return set_error(SAL_ERR_INVALID_ARG, "winding buffer given with SAL_WINDING_NONE");
    if (n > 0 && (!x || !y || !z || !labels))
        return set_error(SAL_ERR_INVALID_ARG, "NULL point or label buffer");
    if (stats) std::memset(stats, 0, sizeof(*stats));
    if (n == 0) return SAL_OK;
    SAL_HIP(hipSetDevice(ctx->device));
    // every argument is checked before anything is enqueued
    if (opt.cull_bounds && (st = ensure_surface_balls(ctx, set)) != SAL_OK) return st;
    if ((st = ensure_label_scratch(ctx, set, n)) != SAL_OK) return st;
    // (without stats nothing reads the counters)
    if (stats) SAL_HIP(launch_fill_u64(ctx->counters, 0ull, kNumCounters, ctx->stream));
    int shape[2] = {0, 0};
    st = enqueue_label(ctx, set, n, x, y, z, opt, labels, winding, stats ? ctx->ev[0] : nullptr,
                       stats ? ctx->ev[1] : nullptr, shape);
    if (st != SAL_OK) return st;
    if (stats) {
        SAL_HIP(hipEventRecord(ctx->ev[2], ctx->stream));
        SAL_HIP(hipEventSynchronize(ctx->ev[2]));
        unsigned long long c[kNumCounters];
        SAL_HIP(hipMemcpy(c, ctx->counters, sizeof(c), hipMemcpyDeviceToHost));
        stats->n_points = n;
        stats->n_pairs = n * set->n_tri;
        stats->n_recheck_points = (int64_t)c[kCntFlagged];
        stats->n_recheck_pairs = (int64_t)c[kCntRecheck];
        stats->n_band_flags = (int64_t)c[kCntBand];
        stats->n_cond_flags = (int64_t)c[kCntCond];
        stats->n_exact_fallbacks = (int64_t)c[kCntExact];
        stats->n_recheck_f64_terms = (int64_t)c[kCntRecheckF64];
        stats->n_pairs_culled = (int64_t)c[kCntCulled];
        SAL_HIP(hipEventElapsedTime(&stats->ms_pairloop, ctx->ev[0], ctx->ev[1]));
        SAL_HIP(hipEventElapsedTime(&stats->ms_total, ctx->ev[0], ctx->ev[2]));
        stats->ms_recheck = stats->ms_total - stats->ms_pairloop;
        stats->points_per_lane = shape[0];
        stats->block_waves = shape[1];
    }
    return SAL_OK;
    SAL_GUARD_END
}

}  // extern "C"

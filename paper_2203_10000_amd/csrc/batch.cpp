// sal_label_batch: many independent (surface set, point set) instances in one
// launch sequence, optionally captured in a hipGraph and replayed.
#include <algorithm>
#include <cstring>
#include <vector>

#include "runtime.h"

namespace sal {
namespace {

// One wavefront a workgroup: its place is free as soon as it ends (four: 24
// instances 1141 us instead of 1080, 8 in fp64 213 instead of 202).
constexpr int kBlockWaves = 1;

template <typename T>
sal_status ensure_dev(T **p, int64_t *have, int64_t need, sal_context *ctx) {
    if (need <= *have) return SAL_OK;
    SAL_HIP(hipStreamSynchronize(ctx->stream));
    if (*p) SAL_HIP(hipFree(*p));
    *p = nullptr;
    *have = 0;
    ctx->batch_graph_fields.clear();   // buffers moved: a captured graph is stale
    const int64_t cap = need + need / 4 + 64;
    SAL_HIP(dev_malloc((void **)p, (size_t)cap * sizeof(T)));
    *have = cap;
    return SAL_OK;
}

bool same_table(const std::vector<LabelInst> &a, const std::vector<LabelInst> &b) {
    return a.size() == b.size() && std::memcmp(a.data(), b.data(), a.size() * sizeof(LabelInst)) == 0;
}

}  // namespace
}  // namespace sal

using namespace sal;

extern "C" sal_status sal_label_batch(sal_context *ctx, const sal_instance *inst, int32_t n_inst,
                                      const sal_label_options *opt_in, sal_label_stats *stats) {
    try {
        if (!ctx || (n_inst > 0 && !inst)) return set_error(SAL_ERR_INVALID_ARG, "NULL argument");
        if (n_inst < 0) return set_error(SAL_ERR_INVALID_ARG, "n_inst < 0");
        sal_label_options opt;
        sal_status st = resolve_options(opt_in, &opt);
        if (st != SAL_OK) return st;
        if (opt.winding_type != SAL_WINDING_NONE)
            return set_error(SAL_ERR_INVALID_ARG, "the batched form has no winding output");
        int64_t total = 0;
        std::vector<int64_t> sizes;
        for (int i = 0; i < n_inst; ++i) {
            const sal_instance &in = inst[i];
            if (!in.surfaces) return set_error(SAL_ERR_INVALID_ARG, "instance without surfaces");
            if (in.surfaces->device != ctx->device)
                return set_error(SAL_ERR_INVALID_ARG, "instance surfaces on another device");
            if (in.n_points < 0) return set_error(SAL_ERR_INVALID_ARG, "n_points < 0");
            if (in.n_points > 0 && (!in.x || !in.y || !in.z || !in.labels))
                return set_error(SAL_ERR_INVALID_ARG, "NULL point or label buffer");
            total += in.n_points;
            sizes.push_back(in.n_points);
        }
        if (stats) std::memset(stats, 0, sizeof(sal_label_stats) * (size_t)n_inst);
        if (total == 0) return SAL_OK;
        SAL_HIP(hipSetDevice(ctx->device));
        hipStream_t s = ctx->stream;

        const bool fp64 = opt.precision == SAL_PREC_FP64;
        if ((st = ensure_dev(&ctx->batch_counters, &ctx->batch_counters_n,
                             (int64_t)n_inst * kNumCounters, ctx)) != SAL_OK)
            return st;

        // The table: the instances of the 64-point form, cut into pieces of at
        // most kChunkPoints, then those labeled point by point.
        std::vector<LabelInst> table;
        ScratchSize need;
        int64_t wave_groups = 0, point_groups = 0;
        size_t n_wave = 0;
        const int64_t point_max = batch_point_max(sizes);
        for (const bool small : {false, true}) {
            for (int i = 0; i < n_inst; ++i) {
                const sal_instance &in = inst[i];
                if ((in.n_points <= point_max) != small) continue;
                for (int64_t at = 0; at < in.n_points; at += kChunkPoints) {
                    const int64_t m = std::min(in.n_points - at, kChunkPoints);
                    LabelInst q = make_inst(in.surfaces, m, in.x + at, in.y + at, in.z + at, in.labels + at,
                                            nullptr, 0, nullptr, ctx->batch_counters + (int64_t)i * kNumCounters);
                    if (small) {
                        q.group_base = point_groups;
                        point_groups += m;
                    } else {
                        q.group_base = wave_groups;
                        q.order_base = need.points;
                        q.tile_base = need.tiles;
                        q.span_entry = need.spans;
                        q.pair_base = need.pairs;
                        wave_groups += group_count(m);
                        need.points += m;
                        need.tiles += q.n_tiles;
                        need.spans += span_count(m) * q.n_surf;
                        need.pairs += group_count(m) * q.n_surf;
                        need.insts += 1;
                    }
                    table.push_back(q);
                }
            }
            if (!small) n_wave = table.size();
        }
        if ((st = ensure_label_scratch(ctx, need)) != SAL_OK) return st;
        if ((int64_t)table.size() > ctx->batch_insts_cap) ctx->batch_table.clear();
        if ((st = ensure_dev(&ctx->batch_insts, &ctx->batch_insts_cap, (int64_t)table.size(), ctx)) != SAL_OK)
            return st;
        if (!same_table(table, ctx->batch_table)) {
            // a graph captured for another batch reads this table, and the
            // previous call may still do so
            ctx->batch_graph_fields.clear();
            ctx->batch_table.clear();
            SAL_HIP(hipStreamSynchronize(s));
            SAL_HIP(hipMemcpy(ctx->batch_insts, table.data(), table.size() * sizeof(LabelInst),
                              hipMemcpyHostToDevice));
            ctx->batch_table = table;
        }

        const LabelScratch sc = context_scratch(ctx);
        LabelArgs a{};
        a.threshold = opt.threshold;
        a.band = opt.recheck_band;
        a.kappa = (float)opt.kappa;
        a.flag_list = sc.flag_list;
        a.work = sc.work;
        a.open_spans = sc.open_spans;
        a.pairs = sc.pairs;
        a.n_pairs = need.pairs;
        a.ord = sc.ord;
        if (need.pairs * 64 >= kSpanPairs) a.span_w = sc.span_w;
        auto enqueue = [&](hipStream_t q) -> sal_status {
            SAL_HIP(launch_fill_u64(ctx->batch_counters, 0ull, (int64_t)n_inst * kNumCounters, q));
            if (n_wave > 0) {
                a.insts = ctx->batch_insts;
                a.n_inst = (int32_t)n_wave;
                SAL_HIP(launch_order(a, need.tiles, q));
                if (a.span_w) SAL_HIP(launch_label_span(a, need.spans, q));
                SAL_HIP(launch_label_pair(a, fp64, std::min<int64_t>(need.pairs, (int64_t)ctx->n_cu * kPairWaves),
                                          kBlockWaves, q));
                SAL_HIP(launch_label_final(a, fp64, wave_groups, q));
            }
            if (point_groups > 0) {
                LabelArgs p = a;
                p.insts = ctx->batch_insts + n_wave;
                p.n_inst = (int32_t)(table.size() - n_wave);
                SAL_HIP(launch_label_point(p, fp64, false, point_groups, kBlockWaves, q));
            }
            if (n_wave > 0) SAL_HIP(launch_recheck(a, fp64, ctx->n_cu * 8, q));
            return SAL_OK;
        };

        // everything the captured launches read or are shaped by
        std::vector<uint64_t> fields(table.size() * (sizeof(LabelInst) / 8));
        static_assert(sizeof(LabelInst) % 8 == 0, "the table is compared as words");
        std::memcpy(fields.data(), table.data(), table.size() * sizeof(LabelInst));
        auto add = [&](const void *p, size_t bytes) {
            uint64_t v = 0;
            std::memcpy(&v, p, bytes);
            fields.push_back(v);
        };
        add(&opt.kappa, 8);
        add(&opt.threshold, 8);
        add(&opt.recheck_band, 8);
        add(&opt.precision, 4);
        add(&n_inst, 4);
        const void *ptrs[] = {ctx->batch_insts, ctx->batch_counters, sc.flag_list, sc.work, sc.ord.idx1,
                              sc.ord.key1, sc.ord.perm, sc.ord.hist, sc.ord.tot, sc.span_w,
                              sc.open_spans, sc.pairs};
        for (const void *p : ptrs) add(&p, sizeof(p));
        const bool replay = opt.use_graph && ctx->batch_graph && ctx->batch_graph_fields == fields;

        if (stats) SAL_HIP(hipEventRecord(ctx->ev[0], s));
        if (opt.use_graph) {
            if (!replay) {
                if (ctx->batch_graph) {
                    SAL_HIP(hipGraphExecDestroy(ctx->batch_graph));
                    ctx->batch_graph = nullptr;
                }
                ctx->batch_graph_fields.clear();
                hipGraph_t g = nullptr;
                SAL_HIP(hipStreamBeginCapture(ctx->capture_stream, hipStreamCaptureModeThreadLocal));
                sal_status cst = enqueue(ctx->capture_stream);
                hipError_t ee = hipStreamEndCapture(ctx->capture_stream, &g);
                if (cst != SAL_OK) {
                    if (g) (void)hipGraphDestroy(g);
                    return cst;
                }
                if (ee != hipSuccess) return hip_error(ee, "hipStreamEndCapture");
                ee = hipGraphInstantiate(&ctx->batch_graph, g, nullptr, nullptr, 0);
                (void)hipGraphDestroy(g);
                if (ee != hipSuccess) return hip_error(ee, "hipGraphInstantiate");
                ctx->batch_graph_fields = fields;
            }
            SAL_HIP(hipGraphLaunch(ctx->batch_graph, s));
        } else {
            if ((st = enqueue(s)) != SAL_OK) return st;
        }
        if (stats) {
            SAL_HIP(hipEventRecord(ctx->ev[2], s));
            SAL_HIP(hipEventSynchronize(ctx->ev[2]));
            float ms = 0.0f;
            SAL_HIP(hipEventElapsedTime(&ms, ctx->ev[0], ctx->ev[2]));
            std::vector<unsigned long long> c((size_t)n_inst * kNumCounters);
            SAL_HIP(hipMemcpy(c.data(), ctx->batch_counters, c.size() * sizeof(unsigned long long),
                              hipMemcpyDeviceToHost));
            for (int i = 0; i < n_inst; ++i) {
                const unsigned long long *ci = c.data() + (size_t)i * kNumCounters;
                stats[i].n_points = inst[i].n_points;
                stats[i].n_pairs = inst[i].n_points * inst[i].surfaces->n_tri;
                stats[i].n_recheck_points = (int64_t)ci[kCntFlagged];
                stats[i].n_recheck_pairs = (int64_t)ci[kCntRecheck];
                stats[i].n_band_flags = (int64_t)ci[kCntBand];
                stats[i].n_cond_flags = (int64_t)ci[kCntCond];
                stats[i].n_exact_fallbacks = (int64_t)ci[kCntExact];
                stats[i].n_recheck_f64_terms = (int64_t)ci[kCntRecheckF64];
                stats[i].ms_total = ms;   // the whole batch (one launch sequence)
                stats[i].ms_pairloop = ms;
                stats[i].points_per_lane = 1;
                stats[i].block_waves = kBlockWaves;
            }
        }
        return SAL_OK;
    } catch (const std::bad_alloc &) {
        return set_error(SAL_ERR_OUT_OF_MEMORY, "host allocation failed");
    } catch (...) {
        return set_error(SAL_ERR_INTERNAL, "exception in sal_label_batch");
    }
}

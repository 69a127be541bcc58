// Surface-set construction: the records, patch trees and leaf boxes that
// surface_host.cpp builds, on the device; the balls of cull_bounds.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <atomic>
#include <vector>

#include "runtime.h"
#include "surface_host.h"

namespace sal {

sal_status build_surface_set(sal_context *ctx, const sal_surface_desc *desc, int32_t n,
                             uint32_t flags, sal_surface_set **out) {
    if (!ctx || !desc || !out) return set_error(SAL_ERR_INVALID_ARG, "NULL argument");
    SurfaceRecords rec;
    sal_status st0 = build_surface_records(desc, n, flags, &rec);
    if (st0 != SAL_OK) return st0;
    const std::vector<SurfaceDev> &table = rec.table;
    const int64_t total_tri = rec.total_tri;
    SAL_HIP(hipSetDevice(ctx->device));
    static std::atomic<uint64_t> next_uid{1};
    auto *set = new sal_surface_set();
    set->uid = next_uid++;
    set->device = ctx->device;
    set->n_surf = n;
    set->n_tri = total_tri;
    set->n_strips = rec.n_leaves;
    set->host_table = table;
    for (int c = 0; c < 3; ++c) {
        set->lo[c] = INFINITY;
        set->hi[c] = -INFINITY;
        for (const SurfaceDev &sd : table) {
            set->lo[c] = std::min(set->lo[c], sd.lo[c]);
            set->hi[c] = std::max(set->hi[c], sd.hi[c]);
        }
    }
    sal_status st = SAL_OK;
    auto up = [&](void **dst, const void *src, size_t bytes) -> sal_status {
        hipError_t e = dev_malloc(dst, bytes);
        if (e != hipSuccess) return hip_error(e, "hipMalloc(surface set)");
        e = hipMemcpy(*dst, src, bytes, hipMemcpyHostToDevice);
        if (e != hipSuccess) return hip_error(e, "hipMemcpy(surface set)");
        set->bytes += bytes;
        return SAL_OK;
    };
    if ((st = up((void **)&set->rec, rec.recs.data(), rec.recs.size() * sizeof(TriRec))) != SAL_OK ||
        (st = up((void **)&set->surf, table.data(), table.size() * sizeof(SurfaceDev))) != SAL_OK ||
        (st = up((void **)&set->ent, rec.entries.data(), rec.entries.size() * sizeof(PatchEntry))) != SAL_OK ||
        (st = up((void **)&set->leaf, rec.leaves.data(), rec.leaves.size() * sizeof(LeafBox))) != SAL_OK) {
        destroy_surface_set(set);
        return st;
    }
    *out = set;
    return SAL_OK;
}

sal_status ensure_surface_balls(sal_context *ctx, const sal_surface_set *cset) {
    auto *set = const_cast<sal_surface_set *>(cset);
    if (set->balls_ready) return SAL_OK;
    const int n = set->n_surf;
    std::vector<SurfaceDev> table = set->host_table;
    std::vector<float> c(3 * (size_t)n);
    for (int i = 0; i < n; ++i)
        for (int a = 0; a < 3; ++a) c[(size_t)(a * n + i)] = table[(size_t)i].ball[a];
    float *dc = nullptr;
    int32_t *dl = nullptr;
    unsigned long long *dm = nullptr;
    std::vector<unsigned long long> masks((size_t)n, 0);
    hipError_t e = dev_malloc((void **)&dc, c.size() * sizeof(float));
    if (e == hipSuccess) e = dev_malloc((void **)&dl, (size_t)n * sizeof(int32_t));
    if (e == hipSuccess) e = dev_malloc((void **)&dm, (size_t)n * sizeof(unsigned long long));
    if (e == hipSuccess) e = hipMemcpy(dc, c.data(), c.size() * sizeof(float), hipMemcpyHostToDevice);
    // each centre against its own surface only: one FP64 launch per surface
    for (int i = 0; i < n && e == hipSuccess; ++i) {
        LabelArgs a{};
        a.one = make_inst(set, 1, dc + i, dc + n + i, dc + 2 * n + i, dl + i, nullptr, 1, dm + i, ctx->counters);
        a.one.surf = set->surf + i;
        a.one.n_surf = 1;
        a.kappa = 0.03125f;
        a.threshold = 0.5;
        a.band = 0.0;
        e = launch_label_point(a, true, false, 1, 1, ctx->stream);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e == hipSuccess) e = hipMemcpy(masks.data(), dm, (size_t)n * sizeof(unsigned long long), hipMemcpyDeviceToHost);
    if (dc) (void)hipFree(dc);
    if (dl) (void)hipFree(dl);
    if (dm) (void)hipFree(dm);
    if (e != hipSuccess) return hip_error(e, "surface ball centres");
    for (int i = 0; i < n; ++i) {
        SurfaceDev &sd = table[(size_t)i];
        sd.ball_w = sd.ball[3] > 0.0f ? (int32_t)(masks[(size_t)i] & 1ull) : -1;
    }
    e = hipMemcpy(set->surf, table.data(), (size_t)n * sizeof(SurfaceDev), hipMemcpyHostToDevice);
    if (e != hipSuccess) return hip_error(e, "hipMemcpy(surface table)");
    set->host_table = table;
    set->balls_ready = true;
    return SAL_OK;
}

void destroy_surface_set(sal_surface_set *set) {
    if (!set) return;
    (void)hipSetDevice(set->device);
    if (set->rec) (void)hipFree(set->rec);
    if (set->surf) (void)hipFree(set->surf);
    if (set->ent) (void)hipFree(set->ent);
    if (set->leaf) (void)hipFree(set->leaf);
    delete set;
}

}  // namespace sal

// Internal declarations shared by the host runtime (*.cpp) and the gfx950
// kernels (*.hip) of libsal.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "sal.h"

namespace sal {

// ---------------------------------------------------------------- records
// A surface is stored as separate triangles (A, B, C), counter-clockwise seen
// from outside, 48 bytes each, so that a lane reads one with three 16-byte loads
// and needs no neighbour:
//   { A, 32 nx, B, 32 ny, C, 32 nz }
// n = (B - A) x (C - A), computed in double from the float32 vertices and
// rounded once.  The factor 32 is a power of two (exact) that folds the
// small-angle bound |N/D| < 1/32 into one comparison.
struct alignas(16) TriRec {
    float v[12];
};

// |N - N_exact| <= ~10 eps |c| |B - A||C - A| for the double triple product
// N = (C - p) . n; a sign is taken as certain above 32 eps |c| |B - A||C - A|
// (32 eps = 2^-48, margin included).
constexpr double kGuardEps = 32.0 * 1.1102230246251565e-16;
constexpr float kNScale = 32.0f;     // normal pre-scale of the records (a power of two)
constexpr float kKnSmall = 5.0f;     // small-angle path needs D > 5 |n| r_C + ...
constexpr int kMaxSurfaces = 64;     // per-point masks are 64-bit

// Patch tree.  The triangles of a surface are grouped into spatially compact
// patches, four to a node, down to leaves of at most kLeafTri triangles.  A
// patch with the opposite of any other surface over the same boundary loops (a
// "cap") is closed, and a closed surface has winding number 0 at every point
// outside its convex hull; so for a point outside the patch's box the cap's
// solid angle equals the patch's.  A cap zigzags over each boundary loop: about
// 3.2 sqrt(m) triangles for a patch of m.  Caps lie inside the
// patch's hull, and the box is enlarged by kCapMargin of its extent, so a point
// outside it sees no cap triangle from close by (float32 certifies the terms).
// Entry e of node w is ent[4 w + e]; an unused entry has leaf_n = 0.
struct alignas(16) PatchEntry {
    float lo[3];
    uint32_t cap_begin;    // the cap: records [cap_begin, cap_begin + cap_n)
    float hi[3];           // box of the patch's vertices, enlarged
    uint32_t cap_n;
    int32_t child;         // node of the patch's parts, -1 for a leaf
    uint32_t leaf_begin;   // the patch's own triangles: records
    uint32_t leaf_n;       // [leaf_begin, leaf_begin + leaf_n)
    uint32_t pad;
};
// Record indices are relative to the surface's rec_begin, node indices to its
// node_begin.

// Leaf size: the lanes of one wavefront.
constexpr int kLeafTri = 64;
constexpr double kCapMargin = 0.02;

// A leaf patch: its triangles' box and records [begin, begin + count); or a group of
// kLeafGroup leaves that follow each other: their box (begin, count: the leaves).
struct alignas(16) LeafBox {
    float lo[3];
    uint32_t begin;
    float hi[3];
    uint32_t count;
};
constexpr int kLeafGroup = 64;

// Per-surface table in device memory.
struct SurfaceDev {
    int64_t rec_begin, rec_end;      // the surface's triangles: records [begin, end)
                                     // (its caps follow)
    int64_t node_begin;              // root node of the patch tree
    int64_t n_tri;
    int64_t leaf_begin;              // its leaves' boxes, then those of their groups
    int32_t label;
    int32_t n_leaves;
    float lo[3], hi[3];              // bounding box of the vertices
    float ball[4];                   // centre and squared radius of a ball the surface does
                                     // not cross (radius shrunk for rounding)
    int32_t ball_w;                  // winding number inside that ball (0 or 1), -1: none
    int32_t pad2;
};

// A point with at least one (surface) winding number that the float32 pass
// cannot certify.
struct FlagEntry {
    uint32_t idx;    // point index within its instance
    int32_t inst;    // instance
    uint64_t enc;    // bit k: float32 pass found w_k >= T
    uint64_t flg;    // bit k: surface k must be recomputed
};

// Device counters (uint64) of one labeling call.
enum Counter {
    kCntFlagged = 0,   // points with a recomputed surface
    kCntBand = 1,      // (point, surface) pairs flagged by the band
    kCntCond = 2,      // pairs flagged by ill-conditioned triangles
    kCntExact = 3,     // exact-sign evaluations
    kCntRecheck = 4,   // pairs recomputed
    kCntRecheckF64 = 5,  // triangle terms of recomputed pairs evaluated in double
    kCntCulled = 6,      // pairs skipped by cull_bounds
    kNumCounters = 8
};

// One set of points against one surface set, as the kernels see it.
struct LabelInst {
    const TriRec *rec;
    const SurfaceDev *surf;
    const PatchEntry *ent;
    const LeafBox *leaf;
    const float *x, *y, *z;
    int32_t *labels;
    void *winding;                // [n_surf][wstride] float or double, or null
    unsigned long long *masks;    // [n] enclosure bits per point, or null
    unsigned long long *counters; // kNumCounters
    int64_t n, wstride;
    int64_t order_base;           // first entry in the spatial order
    int64_t group_base;           // first group of 64 points (or point) in the grids
    int64_t pair_base;            // first (group, surface) pair
    int64_t tile_base;            // first tile of the spatial order
    int64_t span_entry;           // first (span, surface) pair, a span being 8 groups
    int32_t n_tiles, tile;        // tiles of `tile` points
    int32_t n_surf;
    int32_t pad;
    float lo[3], scale[3];        // cells of the spatial order: (p - lo) * scale
};

// Spatial order of the points (order.hip): two stable counting passes over the
// place on a Hilbert curve, kOrderBits1 low bits first.
constexpr int kOrderBits1 = 11, kOrderBits2 = 10;   // 7 bits per axis
constexpr int kOrderBins = 1 << kOrderBits1;
constexpr int64_t kMinTile = 1024, kMaxTiles = 1024;   // per instance

// Points of a span: the groups that may share one winding number.
constexpr int64_t kSpanGroups = 8, kSpanPoints = 64 * kSpanGroups;
constexpr int32_t kSpanUnknown = INT32_MIN;

// What k_label_pair finds for the 64 points of a group against one surface.
struct alignas(16) PairBits {
    uint64_t in;     // winding number >= T
    uint64_t redo;   // to be summed again (not certain, near T, or too far apart)
};

// Device counters of one launch sequence, cleared by launch_order.
enum Work { kWorkFlagged = 0, kWorkOpen = 1, kNumWork = 2 };

struct OrderScratch {
    uint32_t *idx1;   // [points] order after the first pass
    uint16_t *key1;   // [points] the second pass's digits in that order
    uint32_t *perm;   // [points] the order
    uint32_t *hist;   // [tiles][kOrderBins], bin-major within an instance
    uint32_t *tot;    // [instances][kOrderBins]
};

struct LabelArgs {
    LabelInst one;            // the instance when insts is null
    const LabelInst *insts;
    int32_t n_inst;
    int32_t winding_type;
    const int64_t *n_dev;     // when set, the one instance's point count is read here
    int64_t n_dev_skip;       // (less this many, labeled before); one.n is the capacity
                              // that the grids were sized for
    double threshold, band;
    float kappa;
    int32_t cull;             // skip a surface for points strictly outside its box
                              // (w = 0 exactly) or inside its ball (w = ball_w exactly)
    FlagEntry *flag_list;     // capacity: the points
    unsigned long long *work; // kNumWork
    PairBits *pairs;          // (group, surface)
    int64_t n_pairs;          // over all instances
    int32_t *span_w;          // (span, surface): the winding number that all of the span's points
                              // have, or kSpanUnknown; null: no span pass
    uint32_t *open_spans;     // the unknown ones
    OrderScratch ord;
};

__device__ __forceinline__ int64_t label_count(const LabelArgs &a, const LabelInst &in) {
    if (!a.n_dev) return in.n;
    const int64_t n = *a.n_dev - a.n_dev_skip;
    return n < 0 ? 0 : (n < in.n ? n : in.n);
}

// Kernel launchers (label.hip, order.hip); `groups`, `tiles` and `entries` are
// totals over the instances, block_waves the wavefronts of a workgroup.
// Spatial order of every instance's points; also clears a.work.
hipError_t launch_order(const LabelArgs &a, int64_t tiles, hipStream_t s);
// Winding numbers of whole spans, into a.span_w (entries: spans x surfaces).
hipError_t launch_label_span(const LabelArgs &a, int64_t entries, hipStream_t s);
// The open (group, surface) pairs, 64 points of the order per wavefront; `waves`
// wavefronts share them.
hipError_t launch_label_pair(const LabelArgs &a, bool fp64, int64_t waves, int block_waves, hipStream_t s);
// Labels, masks and the flag list from the pairs and spans.
hipError_t launch_label_final(const LabelArgs &a, bool fp64, int64_t groups, hipStream_t s);
// One point per wavefront, no order; results are final (nothing is flagged).
// spread: the surfaces of a point are dealt to the workgroup's wavefronts.
hipError_t launch_label_point(const LabelArgs &a, bool fp64, bool spread, int64_t groups, int block_waves,
                              hipStream_t s);
// Sums the flagged (point, surface) pairs again, one point per wavefront.
hipError_t launch_recheck(const LabelArgs &a, bool fp64, int blocks, hipStream_t s);
hipError_t launch_fill_u64(unsigned long long *p, unsigned long long v, int64_t n, hipStream_t s);

// ------------------------------------------------------------ host helpers
sal_status set_error(sal_status s, const std::string &msg);

// Every device allocation of the library goes through here: hipMalloc, or a
// simulated out-of-memory when sal_debug_fail_allocation armed this call.
hipError_t dev_malloc(void **ptr, size_t bytes);
void fail_allocation(int64_t n);
sal_status hip_error(hipError_t e, const char *what);

// Allocations of meshes and of single calls, from blocks kept on the current
// device (devmem.cpp).  `token` names the stream order that the block is used in
// (sal_context::stream_token); a freed block may still be in use there.  Token 0:
// no work on it is pending.
hipError_t pool_malloc(void **ptr, size_t bytes, uint64_t token);
void pool_free(void *ptr, uint64_t token);
// Waits for the device: what was freed before has no work pending then.
hipError_t pool_device_synchronize();
uint64_t new_stream_token();
void pool_add_context();
void pool_remove_context(uint64_t token);

}  // namespace sal

#define SAL_HIP(expr)                                             \
    do {                                                          \
        hipError_t _e = (expr);                                   \
        if (_e != hipSuccess) return ::sal::hip_error(_e, #expr); \
    } while (0)

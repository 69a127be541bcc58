// Labeling kernels: winding numbers through the patch tree, the label
// decision, and the recomputation of what float32 cannot certify.  gfx950
// (CDNA4), wave64.
//
// Three facts about closed surfaces replace the sum over triangles.  The winding
// numbers of two points differ by the signed number of triangles that the segment
// between them crosses.  They are 0 outside the surface's box, so one segment out
// of it (a ray) gives a point's.  And where no ray is certain, a patch seen from
// outside its box has the solid angle of its cap (see PatchEntry), so the sum takes
// about 8 sqrt(T) terms instead of T.
//   k_label_span   512 neighbouring points (order.hip) and one surface per
//                  wavefront: the winding number they share, if the surface does
//                  not enter their box.
//   k_label_pair   64 neighbouring points and one surface that their span left
//                  open: a ray gives one point of their box its winding number, and
//                  the others differ from it by the signed number of near triangles
//                  that the segment between them crosses.
//   k_label_final  the labels from both.
//   k_label_point  one point per wavefront, a lane per triangle: few points.
//   k_recheck      the same for flagged (point, surface) pairs.
// No MFMA: a term has K = 3 products, square roots and a sign-sensitive sum.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "patch.h"
#include "sal_internal.h"
#include "wave.h"

namespace sal {
namespace {

using patch::Lists;
using patch::Mode;
using patch::PointSum;

// A run of lanes is halved while its box meets too many triangles for the lists,
// down to kSplitMin lanes; below it a ray per point (k_recheck) is cheaper.
// 60,001 points within 1 mm of two surfaces of 162,000 triangles, two shells of
// points of 2,048: 4 lanes 340 and 447 us, 16 lanes 295 and 128, 32 lanes 454 and
// 137.
constexpr int kSplitMin = 16;

// Spans of an instance with fewer points are so large that most meet a surface:
// they are left open unlooked at.  24 instances of up to 353,000 points, two
// rounds under 20 surfaces (us): from 0 points on 1042 and 2616, from 2^16 944 and
// 2597, from 2^18 997 and 2879, from 2^20 1051 and 3711.
constexpr int64_t kSpanInstance = (int64_t)1 << 16;

// Below this many (group, surface) pairs a wavefront takes a quarter of a group:
// its chain is shorter, and the chip has places for all of them.  8,192 pairs or
// fewer (us, whole groups / quarters): 60,001 points by two surfaces 398 / 295;
// 3,072 pairs of 196,608 lattice points 90 / 120.
constexpr int64_t kQuarterPairs = 2048;

// Instance of place g in a grid whose first places the instances hold at BASE.
template <int64_t LabelInst::*BASE>
__device__ __forceinline__ int find_inst(const LabelInst *insts, int n_inst, int64_t g) {
    int lo = 0, hi = n_inst - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (insts[mid].*BASE <= g) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ void store_winding(const LabelInst &in, int type, int k, int64_t i, double w) {
    if (!in.winding) return;
    const int64_t o = (int64_t)k * in.wstride + i;
    if (type == SAL_WINDING_F64) ((double *)in.winding)[o] = w;
    else ((float *)in.winding)[o] = (float)w;
}

// Winding number that cull_bounds gives a point of surface sd without a sum:
// 0 strictly outside the box, the ball's inside it, -1: none.
__device__ __forceinline__ int culled_winding(const SurfaceDev &sd, float x, float y, float z) {
    if (x < sd.lo[0] || x > sd.hi[0] || y < sd.lo[1] || y > sd.hi[1] || z < sd.lo[2] || z > sd.hi[2]) return 0;
    const float dx = x - sd.ball[0], dy = y - sd.ball[1], dz = z - sd.ball[2];
    if (sd.ball_w >= 0 && fmaf(dx, dx, fmaf(dy, dy, dz * dz)) < sd.ball[3]) return sd.ball_w;
    return -1;
}

// One point (the same in every lane) against surface sd: a ray where that is
// certain, else the sum.  A point strictly outside the surface's box is outside
// its convex hull.
template <Mode MODE>
__device__ __forceinline__ PointSum point_surface(const LabelInst &in, const SurfaceDev &sd, Lists &L,
                                                  float x, float y, float z, float kap) {
    if (x < sd.lo[0] || x > sd.hi[0] || y < sd.lo[1] || y > sd.hi[1] || z < sd.lo[2] || z > sd.hi[2])
        return PointSum{0.0, false, 0u, 0u};
    const float p[3] = {x, y, z};
    const TriRec *rec = in.rec + sd.rec_begin;
    const LeafBox *leaf = in.leaf + sd.leaf_begin;
    int v;
    for (int i = 0; i < 2; ++i)
        if (patch::ray_winding(leaf, rec, sd, p, i, L, v)) return PointSum{(double)v, false, 0u, 0u};
    int n_near, n_far;
    if (!patch::sort_patches(in.ent + 4 * sd.node_begin, p, p, L, n_near, n_far)) {
        // A list is full where hundreds of patches share the point: all triangles
        // then, in as many ranges as the list holds, so that every group of lanes has
        // some and a float32 sum stays short (64 points at a vertex of 65,536 triangles,
        // as one range 52 ms, now 8.1).
        const uint32_t all = (uint32_t)(sd.rec_end - sd.rec_begin);
        const uint32_t per = ((all + patch::kNearCap - 1) / patch::kNearCap + 7u) & ~7u;
        n_near = (int)((all + per - 1) / per);
        n_far = 0;
        wave_sync();
        for (uint32_t i = (uint32_t)lane_id(); i < (uint32_t)n_near; i += 64)
            L.near[i] = make_uint2(i * per, all - i * per < per ? all - i * per : per);
        wave_sync();
    }
    const PointSum s = patch::point_sum<MODE>(rec, L, n_near, n_far, x, y, z, kap);
    wave_sync();   // the lists are free again
    return s;
}

// The lanes' boxes joined, in every lane.
__device__ __forceinline__ void box_join(float (&lo)[3], float (&hi)[3]) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            lo[c] = fminf(lo[c], __shfl_xor(lo[c], d));
            hi[c] = fmaxf(hi[c], __shfl_xor(hi[c], d));
        }
        lo[c] = readlane_v(lo[c], 0);
        hi[c] = readlane_v(hi[c], 0);
    }
}

// Box of the points of the lanes with `mine`, in every lane.
__device__ __forceinline__ void box_of(bool mine, float x, float y, float z, float (&lo)[3], float (&hi)[3]) {
    const float inf = __builtin_inff();
    const float p[3] = {x, y, z};
    for (int c = 0; c < 3; ++c) {
        lo[c] = mine ? p[c] : inf;
        hi[c] = mine ? p[c] : -inf;
    }
    box_join(lo, hi);
}

__device__ __forceinline__ void count(unsigned long long *counters, int which, unsigned long long v) {
    if (v && lane_id() == 0) atomicAdd(&counters[which], v);
}

// What single-point sums add to the counters.
struct Tally {
    unsigned exact = 0, n_f64 = 0;            // per lane
    unsigned band = 0, cond = 0, pairs = 0;   // per wavefront
    unsigned points = 0;
    unsigned long long culled = 0;

    __device__ __forceinline__ void flush(unsigned long long *c) {
        const unsigned e = wave_add(exact), f = wave_add(n_f64);
        count(c, kCntExact, e);
        count(c, kCntRecheckF64, f);
        count(c, kCntBand, band);
        count(c, kCntCond, cond);
        count(c, kCntRecheck, pairs);
        count(c, kCntFlagged, points);
        count(c, kCntCulled, culled);
        *this = Tally{};
    }
};

// One point against surface k, final: winding number, enclosure, counters.
// In the float32 form the terms that float32 does not certify are evaluated in
// double on the spot, so such a pair counts as flagged and recomputed.
template <bool F64>
__device__ __forceinline__ bool point_final(const LabelInst &in, const LabelArgs &a, int k, Lists &L, float x,
                                            float y, float z, double &w, Tally &t, bool &flagged) {
    const SurfaceDev &sd = in.surf[k];
    if (a.cull) {
        const int fix = culled_winding(sd, x, y, z);
        if (fix >= 0) {
            t.culled += (unsigned long long)sd.n_tri;
            w = (double)fix;
            return w >= a.threshold;
        }
    }
    const PointSum s = point_surface<F64 ? patch::kDouble : patch::kMixed>(in, sd, L, x, y, z, a.kappa);
    w = s.w;
    t.exact += s.exact;
    if (!F64) {
        t.n_f64 += s.n_f64;
        const bool cond = ballot(s.n_f64 != 0u) != 0, band = fabs(w - a.threshold) < a.band;
        t.cond += cond;
        t.band += band;
        t.pairs += cond || band;
        flagged = flagged || cond || band;
    }
    return s.on || w >= a.threshold;
}

// ------------------------------------------------------------- single points
// What bounds it: latency.  A point costs two dependent loads, of the leaves'
// groups and leaves, and some ten leaves that its ray passes; with one wavefront per
// point (SPREAD: the surfaces dealt to the workgroup's) there is no other serial
// chain.  10,007 points x 4 surfaces of 5,120 triangles: 44 us (as sums over the
// caps 138, a tree level at a time 64).
// Four wavefronts a SIMD (128 VGPRs): with three (133) they take 53 us.
template <bool F64, bool SPREAD>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void k_label_point(LabelArgs a) {
    extern __shared__ __align__(16) unsigned char shared[];
    __shared__ unsigned long long s_enc;
    __shared__ unsigned s_flag;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), waves = (int)(blockDim.x >> 6);
    Lists &L = ((Lists *)shared)[wave];
    const int64_t g = SPREAD ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * waves + wave;
    const int ii = a.insts ? find_inst<&LabelInst::group_base>(a.insts, a.n_inst, g) : 0;
    const LabelInst &in = a.insts ? a.insts[ii] : a.one;
    const int64_t n = label_count(a, in);
    const int64_t i = g - in.group_base;
    const bool live = i < n;
    const float x = live ? in.x[i] : 0.0f, y = live ? in.y[i] : 0.0f, z = live ? in.z[i] : 0.0f;
    const bool good = live && finite3(x, y, z);
    const int lane = lane_id();
    unsigned long long enc = 0;
    Tally t;
    bool flagged = false;
    for (int k = SPREAD ? wave : 0; k < in.n_surf && live; k += SPREAD ? waves : 1) {
        double w = __builtin_nan("");
        if (good && point_final<F64>(in, a, k, L, x, y, z, w, t, flagged)) enc |= 1ull << k;
        if (lane == 0) store_winding(in, a.winding_type, k, i, w);
    }
    if (SPREAD) {
        if (threadIdx.x == 0) { s_enc = 0ull; s_flag = 0u; }
        __syncthreads();
        if (lane == 0 && enc) atomicOr(&s_enc, enc);
        if (lane == 0 && flagged) s_flag = 1u;
        __syncthreads();
        enc = s_enc;
        flagged = s_flag != 0u && wave == 0;
    }
    t.points = flagged;
    if (live && lane == 0 && (!SPREAD || wave == 0)) {
        in.labels[i] = !good ? -1 : enc ? in.surf[63 - __builtin_clzll(enc)].label : 0;
        if (in.masks) in.masks[i] = good ? enc : 0ull;
    }
    t.flush(in.counters);
}

// ------------------------------------------------------------------- spans
// Eight groups share most of their winding numbers: a surface that does not enter
// the box of all 512 points takes one ray here instead of eight.
// One wavefront per (span, surface): with the surfaces of a span one after the
// other the launch was a serial chain (20 surfaces, 660,000 points: 0.33 ms).
// (6M lattice points x 81,920 triangles, all of labeling: 1.79 ms without, 1.19 with.)
// cull_bounds: the winding number that the option's own test gives every point of
// a span.
__device__ __forceinline__ int32_t culled_span(const LabelInst &in, const LabelArgs &a, const SurfaceDev &sd,
                                               int64_t span, int64_t n) {
    bool out = true, ball = sd.ball_w >= 0;
    for (int j = 0; j < (int)kSpanGroups; ++j) {
        const int64_t at = span * kSpanPoints + j * 64 + lane_id();
        if (at >= n) continue;
        const int64_t idx = a.ord.perm[in.order_base + at];
        const float x = in.x[idx], y = in.y[idx], z = in.z[idx];
        if (!finite3(x, y, z)) continue;
        const int w = culled_winding(sd, x, y, z);
        out = out && w == 0;
        ball = ball && w >= 0 && w == sd.ball_w;
    }
    if (ballot(!out) == 0) return 0;
    return ballot(!ball) == 0 ? sd.ball_w : kSpanUnknown;
}

// Entry g: settles it, or returns true where the groups are left to do it.
__device__ __forceinline__ bool span_open(const LabelArgs &a, int64_t g, Lists &L) {
    const int ii = a.insts ? find_inst<&LabelInst::span_entry>(a.insts, a.n_inst, g) : 0;
    const LabelInst &in = a.insts ? a.insts[ii] : a.one;
    const int64_t n = label_count(a, in), span = (g - in.span_entry) / in.n_surf;
    const int k = (int)((g - in.span_entry) % in.n_surf), lane = lane_id();
    if (span * kSpanPoints >= n) return false;
    const float inf = __builtin_inff();
    float lo[3] = {inf, inf, inf}, hi[3] = {-inf, -inf, -inf};
    unsigned long long n_good = 0;
    for (int j = 0; j < (int)kSpanGroups; ++j) {
        const int64_t at = span * kSpanPoints + j * 64 + lane;
        const int64_t idx = at < n ? (int64_t)a.ord.perm[in.order_base + at] : 0;
        const float p[3] = {in.x[idx], in.y[idx], in.z[idx]};
        const bool good = at < n && finite3(p[0], p[1], p[2]);
        n_good += __popcll(ballot(good));
        if (good)
            for (int c = 0; c < 3; ++c) {
                lo[c] = fminf(lo[c], p[c]);
                hi[c] = fmaxf(hi[c], p[c]);
            }
    }
    box_join(lo, hi);
    const SurfaceDev &sd = in.surf[k];
    int32_t v = kSpanUnknown;
    unsigned long long culled = 0;
    if (n < kSpanInstance) {
        // open
    } else if (a.cull && (v = culled_span(in, a, sd, span, n)) != kSpanUnknown) {
        culled = n_good * (unsigned long long)sd.n_tri;
    } else if (!(lo[0] <= hi[0]) || lo[0] > sd.hi[0] || hi[0] < sd.lo[0] || lo[1] > sd.hi[1] || hi[1] < sd.lo[1] ||
        lo[2] > sd.hi[2] || hi[2] < sd.lo[2]) {
        v = 0;
    } else {
        const TriRec *rec = in.rec + sd.rec_begin;
        const LeafBox *leaf = in.leaf + sd.leaf_begin;
        if (patch::triangles_near(leaf, sd.n_leaves, rec, lo, hi, L, 0, 0) == 0) {
            float q[3];
            for (int c = 0; c < 3; ++c) q[c] = 0.5f * lo[c] + 0.5f * hi[c];
            int r;
            if (patch::ray_winding(leaf, rec, sd, q, 0, L, r)) v = r;
        }
    }
    if (lane == 0) a.span_w[g] = v;
    count(in.counters, kCntCulled, culled);
    return v == kSpanUnknown;
}

// The last wavefront of a workgroup lists what all of them left open: the list's
// counter takes some 5 ns an update (us, an update a wavefront, a workgroup of 2, 4
// and 8: 24 instances 944, 914, 909, 916; 6M lattice points 736, 725, 718, 730).
constexpr int kSpanWaves = 4;

__global__ __launch_bounds__(64 * kSpanWaves) void k_label_span(LabelArgs a, int64_t entries) {
    __shared__ Lists lists[kSpanWaves];
    __shared__ uint32_t s_open[kSpanWaves];
    __shared__ unsigned s_n, s_done;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (threadIdx.x == 0) { s_n = 0u; s_done = 0u; }
    __syncthreads();
    const int64_t g = (int64_t)blockIdx.x * kSpanWaves + wave;
    const bool open = g < entries && span_open(a, g, lists[wave]);
    if (lane_id() != 0) return;
    if (open) s_open[atomicAdd(&s_n, 1u)] = (uint32_t)g;
    __threadfence_block();
    if (atomicAdd(&s_done, 1u) != kSpanWaves - 1) return;
    __threadfence_block();
    const unsigned n = s_n;
    if (n == 0) return;
    const unsigned long long base = atomicAdd(&a.work[kWorkOpen], (unsigned long long)n);
    for (unsigned i = 0; i < n; ++i) a.open_spans[base + i] = s_open[i];
}

// ------------------------------------------------------------- open pairs
// What bounds it: the latency of the leaf boxes' and triangles' loads, the crossings,
// some 60 instructions for each triangle that meets the box, and at the launch's end
// the longest wavefronts, whose boxes overflow the lists and are halved.  One
// wavefront per pair: with a group's surfaces one after the other the tail was longer.  The
// point of known winding takes a ray; as a sum over the patches' caps it took 100
// and more rounds of 130 instructions instead of some 10 of 40 (us, sum / ray: 6M
// lattice points x 81,920 triangles 1190 / 820; 60,001 points near two surfaces
// 840 / 420; 24 instances 1650 / 1130).
template <bool F64, int RUNS>
__global__ __launch_bounds__(512) void k_label_pair(LabelArgs a) {
    extern __shared__ __align__(16) unsigned char shared[];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    Lists &L = ((Lists *)shared)[wave];
    const int lane = lane_id();
    typedef typename std::conditional<F64, double, float>::type T;
    const int64_t total = a.span_w ? (int64_t)a.work[kWorkOpen] * kSpanGroups : a.n_pairs * RUNS;
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x >> 6);
    for (int64_t item = (int64_t)blockIdx.x * (blockDim.x >> 6) + wave; item < total; item += waves) {
        int ii = 0, k;
        int64_t group;
        if (RUNS == 1 && a.span_w) {
            const int64_t e = a.open_spans[item / kSpanGroups];
            if (a.insts) ii = find_inst<&LabelInst::span_entry>(a.insts, a.n_inst, e);
            const LabelInst &in = a.insts ? a.insts[ii] : a.one;
            const int64_t r = e - in.span_entry;
            k = (int)(r % in.n_surf);
            group = r / in.n_surf * kSpanGroups + item % kSpanGroups;
        } else {
            const int64_t e = item / RUNS;
            if (a.insts) ii = find_inst<&LabelInst::pair_base>(a.insts, a.n_inst, e);
            const LabelInst &in = a.insts ? a.insts[ii] : a.one;
            const int64_t r = e - in.pair_base;
            k = (int)(r % in.n_surf);
            group = r / in.n_surf;
        }
        const LabelInst &in = a.insts ? a.insts[ii] : a.one;
        const int64_t n = label_count(a, in), at = group * 64 + lane;
        if (group * 64 >= n) continue;
        const SurfaceDev &sd = in.surf[k];
        const int part = RUNS > 1 ? (int)(item % RUNS) : 0, first = part * (64 / RUNS), end = first + 64 / RUNS;
        const bool valid = at < n && lane >= first && lane < end;
        const int64_t idx = valid ? (int64_t)a.ord.perm[in.order_base + at] : 0;
        float px = valid ? in.x[idx] : 0.0f, py = valid ? in.y[idx] : 0.0f, pz = valid ? in.z[idx] : 0.0f;
        const bool good = valid && finite3(px, py, pz);
        if (!good) { px = 0.0f; py = 0.0f; pz = 0.0f; }
        const uint64_t good_mask = ballot(good);
        float lo[3], hi[3];
        box_of(good, px, py, pz, lo, hi);
        double w = 0.0;
        bool cond = false, apart = false;
        bool open = good_mask != 0 && lo[0] <= sd.hi[0] && hi[0] >= sd.lo[0] && lo[1] <= sd.hi[1] &&
                    hi[1] >= sd.lo[1] && lo[2] <= sd.hi[2] && hi[2] >= sd.lo[2];
        if (a.cull && good_mask) {
            const int fix = culled_winding(sd, px, py, pz);
            int same = -1;
            if ((ballot(fix == 0) & good_mask) == good_mask) same = 0;
            else if ((ballot(fix >= 0 && fix == sd.ball_w) & good_mask) == good_mask) same = sd.ball_w;
            if (same >= 0) {
                count(in.counters, kCntCulled,
                      (unsigned long long)__popcll(good_mask) * (unsigned long long)sd.n_tri);
                w = (double)same;
                open = false;
            }
        }
        if (open) {
            const TriRec *rec = in.rec + sd.rec_begin;
            const LeafBox *leaf = in.leaf + sd.leaf_begin;
            // the whole wavefront, or aligned runs of lanes, halved while their box
            // meets more triangles than the lists hold
            for (int pos = first, len = 64 / RUNS; pos < end;) {
                const uint64_t run = (len == 64 ? ~0ull : ((1ull << len) - 1ull) << pos) & good_mask;
                int n_cand = 0, v = 0, delta = 0;
                bool known = false, uncertain = false;
                if (run) {
                    const bool mine = (run >> lane) & 1ull;
                    float blo[3], bhi[3];
                    if (len == 64 / RUNS) {
                        for (int c = 0; c < 3; ++c) { blo[c] = lo[c]; bhi[c] = hi[c]; }
                    } else {
                        box_of(mine, px, py, pz, blo, bhi);
                    }
                    n_cand = patch::triangles_near(leaf, sd.n_leaves, rec, blo, bhi, L, 0, patch::kNearTri);
                    if (n_cand < 0 && len > kSplitMin) {
                        len >>= 1;
                        continue;
                    }
                    // The point of known winding: inside the box, off its planes of
                    // symmetry, so that segments to lattice points seldom pass
                    // through edges of a regular mesh; where one ray does not
                    // settle it, another point.
                    const float frac[3][3] = {{0.4871f, 0.5237f, 0.5113f}, {0.3137f, 0.6719f, 0.4481f},
                                              {0.6863f, 0.3571f, 0.6229f}};
                    for (int i = 0; i < 3 && n_cand >= 0 && !known; ++i) {
                        float q[3];
                        for (int c = 0; c < 3; ++c)
                            q[c] = fminf(fmaxf(fmaf(bhi[c] - blo[c], frac[i][c], blo[c]), blo[c]), bhi[c]);
                        known = patch::ray_winding(leaf, rec, sd, q, i, L, v);
                        if (known && n_cand > 0) {
                            const T d[3] = {(T)px - (T)q[0], (T)py - (T)q[1], (T)pz - (T)q[2]};
                            // (the longest side: where the squares underflow, within the
                            // bounds' factor of two)
                            T d2 = 0, side = 0;
                            for (int c = 0; c < 3; ++c) {
                                const T r = fmax((T)bhi[c] - (T)q[c], (T)q[c] - (T)blo[c]);
                                d2 += r * r;
                                side = fmax(side, r);
                            }
                            patch::near_crossings<T>(rec, L, n_cand, q, d, fmax(sqrt(d2) * (T)1.00001, side),
                                                     delta, uncertain);
                        }
                    }
                }
                if ((run >> lane) & 1ull) {
                    w = (double)(v + delta);
                    cond = known && uncertain;
                    apart = !known;   // left to k_recheck
                }
                pos += len;
                len = pos & -pos;   // the largest run aligned here
            }
        }
        const uint64_t in_bits = ballot(w >= a.threshold) & good_mask;
        uint64_t redo = ballot(apart || cond) & good_mask;
        if (!F64) {
            const uint64_t band = ballot(!apart && fabs(w - a.threshold) < a.band) & good_mask;
            count(in.counters, kCntBand, (unsigned long long)__popcll(band));
            count(in.counters, kCntCond, (unsigned long long)__popcll(ballot(cond) & good_mask));
            redo |= band;
        }
        PairBits *out = a.pairs + in.pair_base + group * in.n_surf + k;
        if (lane == 0 && RUNS == 1) *out = PairBits{in_bits, redo};
        if (lane == 0 && RUNS == 4) {
            ((uint16_t *)&out->in)[part] = (uint16_t)(in_bits >> first);
            ((uint16_t *)&out->redo)[part] = (uint16_t)(redo >> first);
        }
        if (good) store_winding(in, a.winding_type, k, idx, w);
    }
}

// ------------------------------------------------------------------- labels
// Bound by memory: the points are read once more (to find those without a
// place) and the labels written through the order.
template <bool F64>
__global__ __launch_bounds__(256) void k_label_final(LabelArgs a) {
    const int64_t g = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int ii = a.insts ? find_inst<&LabelInst::group_base>(a.insts, a.n_inst, g) : 0;
    const LabelInst &in = a.insts ? a.insts[ii] : a.one;
    const int64_t n = label_count(a, in), group = g - in.group_base;
    const int lane = lane_id();
    const int64_t at = group * 64 + lane;
    if (group * 64 >= n) return;
    const bool valid = at < n;
    const int64_t idx = valid ? (int64_t)a.ord.perm[in.order_base + at] : 0;
    const bool good = valid && finite3(in.x[idx], in.y[idx], in.z[idx]);
    const uint64_t good_mask = ballot(good);
    uint64_t enc = 0, flg = 0;
    int32_t lab = 0;
    unsigned band = 0;
    for (int k = 0; k < in.n_surf; ++k) {
        const int32_t v = a.span_w ? a.span_w[in.span_entry + group / kSpanGroups * in.n_surf + k] : kSpanUnknown;
        bool inside, redo = false;
        if (v != kSpanUnknown) {
            inside = (double)v >= a.threshold;
            redo = !F64 && fabs((double)v - a.threshold) < a.band;
            if (redo) band += (unsigned)__popcll(good_mask);
            if (good) store_winding(in, a.winding_type, k, idx, (double)v);
        } else {
            const PairBits b = a.pairs[in.pair_base + group * in.n_surf + k];
            inside = (b.in >> lane) & 1ull;
            redo = (b.redo >> lane) & 1ull;
        }
        if (inside) { enc |= 1ull << k; lab = in.surf[k].label; }
        if (redo) flg |= 1ull << k;
        if (valid && !good) store_winding(in, a.winding_type, k, idx, __builtin_nan(""));
    }
    if (valid) {
        in.labels[idx] = good ? lab : -1;
        if (in.masks) in.masks[idx] = good ? enc : 0ull;
    }
    const bool want = good && flg != 0;
    const uint64_t m = ballot(want);
    if (m) {
        const int leader = __builtin_ctzll(m);
        int64_t base = 0;
        if (lane == leader) base = (int64_t)atomicAdd(&a.work[kWorkFlagged], (unsigned long long)__popcll(m));
        base = readlane_v(base, leader);
        if (want) {
            FlagEntry e;
            e.idx = (uint32_t)idx;
            e.inst = ii;
            e.enc = enc;
            e.flg = flg;
            a.flag_list[base + lanes_below(m)] = e;
        }
    }
    count(in.counters, kCntBand, band);
}

// Flagged points: their flagged surfaces again, and the label.  A pair's sum
// depends on its point alone, not on its place in the list (the list's order
// is not deterministic).  In the plain FP64 form the list holds the pairs whose
// points were too far apart, and nothing counts as recomputed.
template <bool F64>
__global__ __launch_bounds__(256) void k_recheck(LabelArgs a) {
    __shared__ Lists lists[4];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    Lists &L = lists[wave];
    const int64_t count_n = (int64_t)a.work[kWorkFlagged];
    const int64_t step = (int64_t)gridDim.x * 4;
    const int lane = lane_id();
    Tally t;
    int last = -1;
    for (int64_t j = (int64_t)blockIdx.x * 4 + wave; j < count_n; j += step) {
        const FlagEntry e = a.flag_list[j];
        const int ii = a.insts ? __builtin_amdgcn_readfirstlane(e.inst) : 0;
        const LabelInst &in = a.insts ? a.insts[ii] : a.one;
        if (ii != last && last >= 0) t.flush(a.insts[last].counters);   // (last >= 0 only with insts)
        last = a.insts ? ii : -1;
        const int64_t i = e.idx;
        const float x = in.x[i], y = in.y[i], z = in.z[i];
        unsigned long long enc = e.enc, f = e.flg;
        if (!F64) {
            t.points += 1;
            t.pairs += (unsigned)__popcll(f);
        }
        for (; f; f &= f - 1) {
            const int k = __builtin_ctzll(f);
            const PointSum s = point_surface<F64 ? patch::kDouble : patch::kMixed>(in, in.surf[k], L, x, y, z, a.kappa);
            const double w = s.w;
            t.exact += s.exact;
            t.n_f64 += s.n_f64;
            if (s.on || w >= a.threshold) enc |= 1ull << k;
            else enc &= ~(1ull << k);
            if (lane == 0) store_winding(in, a.winding_type, k, i, w);
        }
        if (lane == 0) {
            in.labels[i] = enc ? in.surf[63 - __builtin_clzll(enc)].label : 0;
            if (in.masks) in.masks[i] = enc;
        }
    }
    if (last >= 0) t.flush(a.insts[last].counters);
    else if (!a.insts) t.flush(a.one.counters);
}

__global__ void k_fill_u64(unsigned long long *p, unsigned long long v, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

}  // namespace

hipError_t launch_label_pair(const LabelArgs &a, bool fp64, int64_t waves, int block_waves, hipStream_t s) {
    if (waves <= 0) return hipSuccess;
    const bool quarters = !a.span_w && a.n_pairs < kQuarterPairs;
    if (quarters) waves = a.n_pairs * 4;
    const dim3 g((unsigned)((waves + block_waves - 1) / block_waves)), b(64u * (unsigned)block_waves);
    const size_t lds = sizeof(Lists) * (size_t)block_waves;
    if (fp64 && quarters) k_label_pair<true, 4><<<g, b, lds, s>>>(a);
    else if (fp64) k_label_pair<true, 1><<<g, b, lds, s>>>(a);
    else if (quarters) k_label_pair<false, 4><<<g, b, lds, s>>>(a);
    else k_label_pair<false, 1><<<g, b, lds, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_label_final(const LabelArgs &a, bool fp64, int64_t groups, hipStream_t s) {
    if (groups <= 0) return hipSuccess;
    const int64_t blocks = (groups + 3) / 4;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    if (fp64) k_label_final<true><<<dim3((unsigned)blocks), dim3(256), 0, s>>>(a);
    else k_label_final<false><<<dim3((unsigned)blocks), dim3(256), 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_label_span(const LabelArgs &a, int64_t entries, hipStream_t s) {
    if (entries <= 0) return hipSuccess;
    if (entries > 0x7fffffff) return hipErrorInvalidValue;
    k_label_span<<<dim3((unsigned)((entries + kSpanWaves - 1) / kSpanWaves)), dim3(64 * kSpanWaves), 0, s>>>(
        a, entries);
    return hipGetLastError();
}

hipError_t launch_label_point(const LabelArgs &a, bool fp64, bool spread, int64_t groups, int block_waves,
                              hipStream_t s) {
    if (groups <= 0) return hipSuccess;
    const int64_t blocks = spread ? groups : (groups + block_waves - 1) / block_waves;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 g((unsigned)blocks), b(64u * (unsigned)block_waves);
    const size_t lds = sizeof(Lists) * (size_t)block_waves;
    if (fp64 && spread) k_label_point<true, true><<<g, b, lds, s>>>(a);
    else if (fp64) k_label_point<true, false><<<g, b, lds, s>>>(a);
    else if (spread) k_label_point<false, true><<<g, b, lds, s>>>(a);
    else k_label_point<false, false><<<g, b, lds, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_recheck(const LabelArgs &a, bool fp64, int blocks, hipStream_t s) {
    if (blocks <= 0) return hipSuccess;
    if (fp64) k_recheck<true><<<dim3((unsigned)blocks), dim3(256), 0, s>>>(a);
    else k_recheck<false><<<dim3((unsigned)blocks), dim3(256), 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_fill_u64(unsigned long long *p, unsigned long long v, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int64_t blocks = (n + 255) / 256;
    k_fill_u64<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(p, v, n);
    return hipGetLastError();
}

}  // namespace sal

// Labeling kernels: winding numbers through the patch tree, the label
// decision, and the recomputation of what float32 cannot certify.  gfx950
// (CDNA4), wave64.
//
// Two facts about closed surfaces replace most of the sum over triangles.  A
// patch seen from outside its box has the solid angle of its cap (see
// PatchEntry), so a point needs about 8 sqrt(T) terms instead of T.  And the
// winding number is constant where the surface does not pass: a wavefront whose
// 64 points lie in a box that meets no triangle needs it at one of them.
//   k_label_wave   64 neighbouring points (order.hip) per wavefront: the
//                  surface is summed at one point of their box, a lane per
//                  triangle, and the others differ from it by the signed number of
//                  near triangles that the segment between them crosses.
//   k_label_point  one point per wavefront, a lane per term: few points.
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

// A run of lanes is halved while its box meets more leaves than this (each costs
// a load, a test of 64 triangles, and ~80 instructions for every triangle that
// meets the box; a halved run sums one point more), down to kSplitMin lanes.
constexpr int kSplitLeaves = 32, kSplitMin = 4;

// Instance of wavefront g, by its place in the grid.
__device__ __forceinline__ int find_group(const LabelInst *insts, int n_inst, int64_t g) {
    int lo = 0, hi = n_inst - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (insts[mid].group_base <= g) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// A closed surface's winding number is a whole number at every point off it:
// the sum's rounding is dropped.  Sums that are not near one (points on the
// surface) are left as they are.
__device__ __forceinline__ double whole(double w) {
    const double r = rint(w);
    return fabs(w - r) < 1e-3 ? r : w;
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

// One point (the same in every lane) against surface sd.  A point strictly
// outside the surface's box is outside its convex hull.
template <Mode MODE>
__device__ __forceinline__ PointSum point_surface(const LabelInst &in, const SurfaceDev &sd, Lists &L,
                                                  float x, float y, float z, float kap) {
    if (x < sd.lo[0] || x > sd.hi[0] || y < sd.lo[1] || y > sd.hi[1] || z < sd.lo[2] || z > sd.hi[2])
        return PointSum{0.0, false, false, 0u, 0u};
    const float p[3] = {x, y, z};
    int n_near, n_far;
    if (!patch::sort_patches(in.ent + 4 * sd.node_begin, p, p, L, n_near, n_far)) {
        // (a list is full only where hundreds of patches share the point)
        n_near = 1;
        n_far = 0;
        wave_sync();
        if (lane_id() == 0) L.near[0] = make_uint2(0u, (uint32_t)(sd.rec_end - sd.rec_begin));
        wave_sync();
    }
    const PointSum s = patch::point_sum<MODE>(in.rec + sd.rec_begin, L, n_near, n_far, x, y, z, kap);
    wave_sync();   // the lists are free again
    return s;
}

// Box of the points of the lanes with `mine`, in every lane.
__device__ __forceinline__ void box_of(bool mine, float x, float y, float z, float (&lo)[3], float (&hi)[3]) {
    const float inf = __builtin_inff();
    const float p[3] = {x, y, z};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        float a = mine ? p[c] : inf, b = mine ? p[c] : -inf;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            a = fminf(a, __shfl_xor(a, d));
            b = fmaxf(b, __shfl_xor(b, d));
        }
        lo[c] = readlane_v(a, 0);
        hi[c] = readlane_v(b, 0);
    }
}

__device__ __forceinline__ unsigned wave_add(unsigned v) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) v += (unsigned)__shfl_xor((int)v, d);
    return v;
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
    w = s.on ? s.half * kInv2Pi : whole(s.half * kInv2Pi);
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
// What bounds it: latency.  A point costs two dependent loads per tree level
// and about 8 sqrt(T) / 64 rounds of triangle loads; with one wavefront per
// point (SPREAD: per point and fourth of its surfaces) there is no other
// serial chain.
template <bool F64, bool SPREAD>
__global__ __launch_bounds__(512) void k_label_point(LabelArgs a) {
    extern __shared__ __align__(16) unsigned char shared[];
    __shared__ unsigned long long s_enc;
    __shared__ unsigned s_flag;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), waves = (int)(blockDim.x >> 6);
    Lists &L = ((Lists *)shared)[wave];
    const int64_t g = SPREAD ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * waves + wave;
    const int ii = a.insts ? find_group(a.insts, a.n_inst, g) : 0;
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

// ------------------------------------------------------------- 64 per wavefront
// What bounds it: load latency in the sum at the box's point and in the tree; the
// crossings are some 80 instructions a triangle that meets the box.  6M lattice
// points x 81,920 triangles, this kernel: 8.0 ms with a lane-by-lane walk over
// the patches where the surface enters the box (1400 terms a point), 3.4 with the
// crossings, 1.9 with one 48-byte record a triangle instead of strips (one
// round of loads a term instead of three), 1.4 in Hilbert instead of Morton order.
template <bool F64>
__global__ __launch_bounds__(512) void k_label_wave(LabelArgs a) {
    extern __shared__ __align__(16) unsigned char shared[];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), waves = (int)(blockDim.x >> 6);
    Lists &L = ((Lists *)shared)[wave];
    const int64_t g = (int64_t)blockIdx.x * waves + wave;
    const int ii = a.insts ? find_group(a.insts, a.n_inst, g) : 0;
    const LabelInst &in = a.insts ? a.insts[ii] : a.one;
    const int64_t n = label_count(a, in);
    const int lane = lane_id();
    const int64_t at = (g - in.group_base) * 64 + lane;
    if (at - lane >= n) return;
    const bool valid = at < n;
    const int64_t idx = valid ? (int64_t)a.ord.perm[in.order_base + at] : 0;
    float px = valid ? in.x[idx] : 0.0f, py = valid ? in.y[idx] : 0.0f, pz = valid ? in.z[idx] : 0.0f;
    const bool good = valid && finite3(px, py, pz);
    if (!good) { px = 0.0f; py = 0.0f; pz = 0.0f; }
    const uint64_t good_mask = ballot(good);
    float lo[3], hi[3];
    box_of(good, px, py, pz, lo, hi);
    uint64_t enc = 0, flg = 0;
    int32_t lab = 0;
    Tally t;
    typedef typename std::conditional<F64, double, float>::type T;
    for (int k = 0; k < in.n_surf; ++k) {
        const SurfaceDev &sd = in.surf[k];
        double w = 0.0;
        bool cond = false, apart = false;
        bool outside = good_mask == 0 || lo[0] > sd.hi[0] || hi[0] < sd.lo[0] || lo[1] > sd.hi[1] ||
                       hi[1] < sd.lo[1] || lo[2] > sd.hi[2] || hi[2] < sd.lo[2];
        if (a.cull && good_mask) {
            const int fix = culled_winding(sd, px, py, pz);
            int same = -1;
            if ((ballot(fix == 0) & good_mask) == good_mask) same = 0;
            else if ((ballot(fix >= 0 && fix == sd.ball_w) & good_mask) == good_mask) same = sd.ball_w;
            if (same >= 0) {
                t.culled += (unsigned long long)__popcll(good_mask) * (unsigned long long)sd.n_tri;
                w = (double)same;
                outside = true;   // settled
            }
        }
        if (!outside) {
            const TriRec *rec = in.rec + sd.rec_begin;
            // the whole wavefront, or aligned runs of lanes, halved while their box
            // meets too many leaves
            for (int pos = 0, len = 64; pos < 64;) {
                const uint64_t run = (len == 64 ? ~0ull : ((1ull << len) - 1ull) << pos) & good_mask;
                float blo[3], bhi[3];
                int n_near = 0, n_far = 0;
                bool fits = true;
                if (run) {
                    if (len == 64) {
                        for (int c = 0; c < 3; ++c) { blo[c] = lo[c]; bhi[c] = hi[c]; }
                    } else {
                        const bool mine = (run >> lane) & 1ull;
                        box_of(mine, px, py, pz, blo, bhi);
                    }
                    fits = patch::sort_patches(in.ent + 4 * sd.node_begin, blo, bhi, L, n_near, n_far);
                    if ((!fits || n_near > kSplitLeaves) && len > kSplitMin) {
                        len >>= 1;
                        wave_sync();
                        continue;
                    }
                }
                double v = 0.0;
                int delta = 0;
                bool known = false, uncertain = false;
                // The sum's point: inside the box, off its planes of symmetry, so
                // that segments to lattice points seldom pass through edges of a
                // regular mesh; where float32 does not certify its sum, another.
                const float at[3][3] = {{0.4871f, 0.5237f, 0.5113f}, {0.3137f, 0.6719f, 0.4481f},
                                        {0.6863f, 0.3571f, 0.6229f}};
                for (int i = 0; i < 3 && run && fits && !known; ++i) {
                    float q[3];
                    for (int c = 0; c < 3; ++c)
                        q[c] = fminf(fmaxf(fmaf(bhi[c] - blo[c], at[i][c], blo[c]), blo[c]), bhi[c]);
                    const PointSum s = patch::point_sum<F64 ? patch::kDouble : patch::kFloat>(
                        rec, L, n_near, n_far, q[0], q[1], q[2], a.kappa);
                    v = rint(s.half * kInv2Pi);
                    known = !s.uncertain && !s.on && fabs(s.half * kInv2Pi - v) < 1e-3;
                    t.exact += s.exact;
                    if (known && n_near > 0) {
                        const T d[3] = {(T)px - (T)q[0], (T)py - (T)q[1], (T)pz - (T)q[2]};
                        T d2 = 0;
                        for (int c = 0; c < 3; ++c) {
                            const T r = fmax((T)bhi[c] - (T)q[c], (T)q[c] - (T)blo[c]);
                            d2 += r * r;
                        }
                        patch::near_crossings<T>(rec, L, n_near, blo, bhi, q, d, sqrt(d2) * (T)1.00001, delta,
                                                 uncertain);
                    }
                }
                if ((run >> lane) & 1ull) {
                    w = v + (double)delta;
                    cond = known && uncertain;
                    apart = !known;   // left to k_recheck
                }
                wave_sync();   // the lists are free again
                pos += len;
                len = pos & -pos;   // the largest run aligned here
            }
        }
        const bool inside = w >= a.threshold;
        if (apart || cond) flg |= 1ull << k;
        if (!F64 && !apart) {
            const bool band = fabs(w - a.threshold) < a.band;
            t.band += __popcll(ballot(band) & good_mask);
            t.cond += __popcll(ballot(cond) & good_mask);
            if (band) flg |= 1ull << k;
        }
        if (inside) { enc |= 1ull << k; lab = sd.label; }
        if (valid) store_winding(in, a.winding_type, k, idx, good ? w : __builtin_nan(""));
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
        if (lane == leader) base = (int64_t)atomicAdd(a.list_n, (unsigned long long)__popcll(m));
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
    t.flush(in.counters);
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
    const int64_t count_n = (int64_t)*a.list_n;
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
            const double w = s.on ? s.half * kInv2Pi : whole(s.half * kInv2Pi);
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

hipError_t launch_label_wave(const LabelArgs &a, bool fp64, int64_t groups, int block_waves, hipStream_t s) {
    if (groups <= 0) return hipSuccess;
    const int64_t blocks = (groups + block_waves - 1) / block_waves;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 g((unsigned)blocks), b(64u * (unsigned)block_waves);
    const size_t lds = sizeof(Lists) * (size_t)block_waves;
    if (fp64) k_label_wave<true><<<g, b, lds, s>>>(a);
    else k_label_wave<false><<<g, b, lds, s>>>(a);
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

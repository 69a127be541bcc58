// Device side of the patch tree: which patches of a surface are near a box,
// and the winding sum of one point by a whole wavefront.
#pragma once

#include <hip/hip_runtime.h>

#include "sal_internal.h"
#include "tri_f64.h"
#include "wave.h"

namespace sal {
namespace patch {

constexpr int kNearCap = 96;    // near leaves of one box (96 x ~45 triangles)
constexpr int kNearTri = 512;   // triangles that may meet a box
constexpr int kRayTri = 256;    // and a ray's box
constexpr int kFarCap = 384;    // far patches: 3 siblings per level and near node
constexpr int kFrontCap = 64;   // near nodes of one level

// One wavefront's working lists in LDS (4.4 KB: 37 wavefronts fit a CU's LDS,
// so they do not limit occupancy).  Patches are record ranges {begin, count},
// triangles record numbers.
struct Lists {
    uint2 near[kNearCap];
    union {
        uint2 far[kFarCap];
        uint32_t tri[kNearTri + kRayTri];
    };
    uint32_t front[2][kFrontCap];
};

// Sorts the surface's patches by the box [lo, hi] (the same in every lane):
// patches whose box it misses go to the far list as their caps, leaves it
// meets to the near list.  Sixteen nodes are opened at a time, one lane per
// entry.  False when a list is full.
__device__ __forceinline__ bool sort_patches(const PatchEntry *__restrict__ ent, const float (&lo)[3],
                                             const float (&hi)[3], Lists &L, int &n_near, int &n_far) {
    const int lane = lane_id();
    int nf = 1, side = 0;
    n_near = 0;
    n_far = 0;
    if (lane == 0) L.front[0][0] = 0u;
    wave_sync();
    while (nf > 0) {
        int nf2 = 0;
        for (int b = 0; b < nf; b += 16) {
            const int i = b + (lane >> 2);
            const bool have = i < nf;
            const uint32_t w = L.front[side][have ? i : 0];
            const uint4 *q = (const uint4 *)(ent + (4ull * w + (lane & 3)));
            const uint4 e0 = q[0], e1 = q[1], e2 = q[2];
            const bool live = have && e2.z != 0u;
            const bool meets = lo[0] <= __uint_as_float(e1.x) && hi[0] >= __uint_as_float(e0.x) &&
                               lo[1] <= __uint_as_float(e1.y) && hi[1] >= __uint_as_float(e0.y) &&
                               lo[2] <= __uint_as_float(e1.z) && hi[2] >= __uint_as_float(e0.z);
            const bool leaf = (int32_t)e2.x < 0;
            const bool to_far = live && !meets && e1.w != 0u;
            const bool to_near = live && meets && leaf;
            const bool open = live && meets && !leaf;
            const uint64_t mf = ballot(to_far), mn = ballot(to_near), mo = ballot(open);
            if (n_far + __popcll(mf) > kFarCap || n_near + __popcll(mn) > kNearCap ||
                nf2 + __popcll(mo) > kFrontCap)
                return false;
            if (to_far) L.far[n_far + lanes_below(mf)] = make_uint2(e0.w, e1.w);
            if (to_near) L.near[n_near + lanes_below(mn)] = make_uint2(e2.y, e2.z);
            if (open) L.front[side ^ 1][nf2 + lanes_below(mo)] = e2.x;
            n_far += __popcll(mf);
            n_near += __popcll(mn);
            nf2 += __popcll(mo);
        }
        wave_sync();
        nf = nf2;
        side ^= 1;
    }
    return true;
}

__device__ __forceinline__ Tri load_tri(const TriRec *__restrict__ rec, uint32_t r) {
    const float4 *q = (const float4 *)(rec + r);
    const float4 a = q[0], b = q[1], c = q[2];
    return Tri{{a.x, a.y, a.z}, {b.x, b.y, b.z}, {c.x, c.y, c.z}, {a.w, b.w, c.w}};
}

// Float32 takes no term whose products are smaller.
constexpr float kLeast = 1e-36f;

struct PointSum {
    double w;          // winding number
    bool on;           // the point lies on a triangle
    unsigned exact;    // exact-sign evaluations, this lane's
    unsigned n_f64;    // float32 terms recomputed in double, this lane's
};

// How a point's terms are evaluated: in float32, those that it does not certify
// in double, or all in double.
enum Mode { kMixed, kDouble };

// A closed surface has a whole winding number at every point off it.
__device__ __forceinline__ double whole(double w) {
    const double r = rint(w);
    return fabs(w - r) < 1e-3 ? r : w;
}

// Winding number of the listed ranges at one point (the same in every lane).
// Eight groups of eight lanes take ranges in turn, a group the next one as it
// becomes free (all lanes run in step, so the assignment, and with it the
// result, depends on the lists alone); a lane evaluates one triangle.  Most
// caps have 20-60 triangles, so wider groups would leave more lanes idle at a
// range's end.  The next triangles are loaded before the present ones are
// evaluated: a round waits for memory only as far as the arithmetic of the
// rounds and of the other wavefronts does not cover it.
template <Mode MODE>
__device__ __forceinline__ PointSum point_sum(const TriRec *__restrict__ rec, const Lists &L, int n_near,
                                              int n_far, float px, float py, float pz, float kap) {
    const int lane = lane_id(), sub = lane & 7;
    const float branch_cut = kPiF - 0.25f * kap;
    const int items = n_near + n_far;
    const uint64_t leaders = 0x0101010101010101ull;
    PointSum out{0.0, false, 0u, 0u};
    float accf = 0.0f;
    double acc = 0.0;
    int next = 0, on = 0;
    uint32_t cur = 0, end = 0;   // this group's range
    bool more = true, cap = false;
    // the lane's triangle of the coming round
    Tri t;
    bool have, t_cap;
    auto fetch = [&]() {
        // groups whose range is finished take the next ones in group order
        const bool need = more && cur >= end;
        const uint64_t m = ballot(need);
        if (m != 0) {
            const int it = next + __popcll(m & leaders & ((1ull << (lane & ~7)) - 1ull));
            if (need) {
                acc += (double)accf;   // (float32 sums end with their range)
                accf = 0.0f;
                more = it < items;
                cap = it >= n_near;
                if (more) {
                    const uint2 g = cap ? L.far[it - n_near] : L.near[it];
                    cur = g.x;
                    end = g.x + g.y;
                }
            }
            next += __popcll(m & leaders);
        }
        const uint32_t r = cur + (uint32_t)sub;
        have = more && r < end;
        t_cap = cap;
        t = load_tri(rec, have ? r : 0u);   // (record 0 exists: the loads are unconditional)
        cur += 8;
    };
    fetch();
    while (ballot(have) != 0) {
        const Tri q = t;
        const bool live = have, q_cap = t_cap;
        fetch();
        if (MODE == kDouble) {
            if (live) {
                const F64Term d = f64_term(q, px, py, pz, q_cap);
                acc += d.half;
                on |= d.on;
                out.exact += d.exact;
            }
            continue;
        }
        const float ax = q.A[0] - px, ay = q.A[1] - py, az = q.A[2] - pz;
        const float bx = q.B[0] - px, by = q.B[1] - py, bz = q.B[2] - pz;
        const float cx = q.C[0] - px, cy = q.C[1] - py, cz = q.C[2] - pz;
        const float ar = __builtin_amdgcn_sqrtf(fmaf(ax, ax, fmaf(ay, ay, az * az)));
        const float br = __builtin_amdgcn_sqrtf(fmaf(bx, bx, fmaf(by, by, bz * bz)));
        const float cr = __builtin_amdgcn_sqrtf(fmaf(cx, cx, fmaf(cy, cy, cz * cz)));
        const float len = __builtin_amdgcn_sqrtf(fmaf(q.n[0], q.n[0], fmaf(q.n[1], q.n[1], q.n[2] * q.n[2])));
        const float e01 = fmaf(ax, bx, fmaf(ay, by, az * bz));
        const float e02 = fmaf(ax, cx, fmaf(ay, cy, az * cz));
        const float e12 = fmaf(bx, cx, fmaf(by, cy, bz * cz));
        const float nn = fmaf(cx, q.n[0], fmaf(cy, q.n[1], cz * q.n[2]));   // 32 N
        const float mm = ar * br * cr;
        const float dd = fmaf(e12, ar, fmaf(e02, br, fmaf(e01, cr, mm)));
        // (kLeast: products that underflow err by far less than 1e-8 of it; a product
        // that overflows certifies nothing)
        const bool finite = fmaxf(fabsf(nn), fabsf(dd)) < __builtin_inff();
        const float lim = fmaf(len * (kKnSmall / kNScale), cr, fmaf(kap, mm, fabsf(nn) + kLeast));
        if (__builtin_expect(live && finite && dd > lim, 1)) {   // |N / D| < 1/32: the series
            const float u = nn * __builtin_amdgcn_rcpf(dd);
            const float s2 = u * u;
            accf = fmaf(u, fmaf(fmaf(kA2, s2, kA1), s2, kA0), accf);
        } else if (live) {
            const float n1 = nn * (1.0f / kNScale);
            const float ang = atan2f(n1, dd);
            const float thr = fmaf(cr, kap * (1.0f / kNScale) * len, fmaf(kap, mm, kLeast));
            const bool ill = !finite || !(fmaxf(fabsf(n1), fabsf(dd)) > thr) || fabsf(ang) > branch_cut;
            if (!ill) {
                accf += ang;
            } else {
                const F64Term d = f64_term(q, px, py, pz, q_cap);
                acc += d.half;
                on |= d.on;
                out.exact += d.exact;
                out.n_f64 += 1u;
            }
        }
    }
    acc += (double)accf;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) acc += __shfl_xor(acc, d);
    out.on = ballot(on != 0) != 0;
    out.w = out.on ? acc * kInv2Pi : whole(acc * kInv2Pi);
    return out;
}

// ----------------------------------------------------------------- crossings
// Winding numbers of 64 points p in a box from that of one point q in it: the
// segment q p stays in the box, and only triangles that meet the box can cross
// it.  A triangle is crossed when p and q lie on different sides of its plane and
// the line passes it on one side of all three edges.  The signs come from
// products relative to q, with bounds on their rounding (u the unit roundoff, L
// the largest distance of a vertex from q, D that of a point): edge products
// err by less than 12 u L^2 D, plane products by less than 10 u |n| (D + L) plus
// the double rounding of n; twice that is taken, and a few of the smallest numbers
// for each product that underflows (`least`).  A lane whose sign is within a bound,
// and not settled by the others, is uncertain.
template <typename T>
struct Bounds;
template <>
struct Bounds<float> {
    static constexpr float edge = 24.0f * 5.9604645e-8f, plane = 20.0f * 5.9604645e-8f;
    static constexpr float normal = 1.5e-13f;   // 32 (scaled normals) x 4.7e-15, per L^2
    static constexpr float huge = 1e37f, least = 1e-44f;
};
template <>
struct Bounds<double> {
    static constexpr double edge = 24.0 * 1.1102230246251565e-16, plane = 20.0 * 1.1102230246251565e-16;
    static constexpr double normal = 5e-15;
    static constexpr double huge = 1e300, least = 0.0;   // (products of float32 numbers)
};

// What 64 points need of one triangle, relative to q.
template <typename T>
struct Crossing {
    T e[3][3];   // edge products (A - q) x (B - q) and on
    T n[3], s;   // side * normal, side * n . (C - q)
    T tol_e, tol_s;
    int side;    // +1: q outside (n . (q - C) > 0), -1: inside, 0: not certain

    __device__ __forceinline__ Crossing from(int lane) const {
        Crossing o;
        for (int i = 0; i < 3; ++i) {
            for (int c = 0; c < 3; ++c) o.e[i][c] = readlane_v(e[i][c], lane);
            o.n[i] = readlane_v(n[i], lane);
        }
        o.s = readlane_v(s, lane);
        o.tol_e = readlane_v(tol_e, lane);
        o.tol_s = readlane_v(tol_s, lane);
        o.side = readlane_i(side, lane);
        return o;
    }
};

__device__ __forceinline__ float fma_t(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return fma(a, b, c); }
template <typename T>
__device__ __forceinline__ T dot_t(const T (&a)[3], const T (&b)[3]) {
    return fma_t(a[0], b[0], fma_t(a[1], b[1], a[2] * b[2]));
}

template <typename T>
__device__ __forceinline__ Crossing<T> make_crossing(const Tri &t, const float (&q)[3], T D) {
    typedef Bounds<T> B;
    Crossing<T> o;
    T v[3][3], l2 = 0, n[3];
    if (sizeof(T) == 8) {
        const T e1[3] = {(T)t.B[0] - (T)t.A[0], (T)t.B[1] - (T)t.A[1], (T)t.B[2] - (T)t.A[2]};
        const T e2[3] = {(T)t.C[0] - (T)t.A[0], (T)t.C[1] - (T)t.A[1], (T)t.C[2] - (T)t.A[2]};
        for (int c = 0; c < 3; ++c) {
            const int u = (c + 1) % 3, w = (c + 2) % 3;
            n[c] = e1[u] * e2[w] - e1[w] * e2[u];
        }
    } else {
        for (int c = 0; c < 3; ++c) n[c] = (T)t.n[c];
    }
    for (int c = 0; c < 3; ++c) {
        v[0][c] = (T)t.A[c] - (T)q[c];
        v[1][c] = (T)t.B[c] - (T)q[c];
        v[2][c] = (T)t.C[c] - (T)q[c];
    }
    for (int i = 0; i < 3; ++i) {
        const T d2 = dot_t(v[i], v[i]);
        l2 = d2 > l2 ? d2 : l2;
        const T(&a)[3] = v[i], (&b)[3] = v[(i + 1) % 3];
        o.e[i][0] = fma_t(a[1], b[2], -(a[2] * b[1]));
        o.e[i][1] = fma_t(a[2], b[0], -(a[0] * b[2]));
        o.e[i][2] = fma_t(a[0], b[1], -(a[1] * b[0]));
    }
    const T len = fabs(n[0]) + fabs(n[1]) + fabs(n[2]), reach = D + sqrt(l2);
    const T s = dot_t(n, v[2]);
    o.tol_e = D * (B::edge * l2 + B::least) + B::least;
    o.tol_s = reach * (B::plane * len + B::normal * l2 + B::least) + B::least;
    // far out of range: nothing is certain, neither a product that overflows (also
    // catches NaN)
    if (!(l2 * reach < B::huge) || !(len * reach < B::huge)) o.tol_e = o.tol_s = (T)__builtin_inf();
    o.side = s < -o.tol_s ? 1 : (s > o.tol_s ? -1 : 0);
    for (int c = 0; c < 3; ++c) o.n[c] = (T)o.side * n[c];
    o.s = (T)o.side * s;
    return o;
}

// Adds the change of the winding number from q to q + d where the triangle is
// crossed (entering: +1).
template <typename T>
__device__ __forceinline__ void cross(const Crossing<T> &t, const T (&d)[3], int &delta, bool &uncertain) {
    const T a = fma_t(t.n[0], d[0], fma_t(t.n[1], d[1], fma_t(t.n[2], d[2], -t.s)));   // > 0: q's side
    const T u = dot_t(t.e[0], d), v = dot_t(t.e[1], d), w = dot_t(t.e[2], d);
    const bool pos = u > t.tol_e && v > t.tol_e && w > t.tol_e, neg = u < -t.tol_e && v < -t.tol_e && w < -t.tol_e;
    const bool beside = (u > t.tol_e || v > t.tol_e || w > t.tol_e) && (u < -t.tol_e || v < -t.tol_e || w < -t.tol_e);
    const bool same = a > t.tol_s, through = a < -t.tol_s;
    if (same || beside) return;
    if (through && (pos || neg)) delta += t.side;
    else uncertain = true;
}

__device__ __forceinline__ void box_terms(const float (&lo)[3], const float (&hi)[3], float (&c)[3], float (&h)[3],
                                          float &scale) {
    scale = 0.0f;
    for (int k = 0; k < 3; ++k) {
        c[k] = 0.5f * lo[k] + 0.5f * hi[k];
        h[k] = 0.5f * hi[k] - 0.5f * lo[k];
        scale += fabsf(c[k]) + h[k];
    }
}

// Whether triangle t may meet the box of centre c and half extents h (scale: |c|
// + h): its own box does (exact comparisons) and its plane passes within the
// box's radius, with a margin some thirty times the products' rounding.  A product
// that overflows excludes nothing; the margin's least terms are for those that
// underflow (in c and h too).
__device__ __forceinline__ bool may_meet(const Tri &t, const float (&lo)[3], const float (&hi)[3],
                                         const float (&c)[3], const float (&h)[3], float scale) {
    bool meets = true;
    float ext = 0.0f;
    for (int k = 0; k < 3; ++k) {
        const float a = fminf(fminf(t.A[k], t.B[k]), t.C[k]), b = fmaxf(fmaxf(t.A[k], t.B[k]), t.C[k]);
        meets = meets && a <= hi[k] && b >= lo[k];
        ext = fmaxf(ext, b - a);
    }
    const float s = fmaf(c[0] - t.C[0], t.n[0], fmaf(c[1] - t.C[1], t.n[1], (c[2] - t.C[2]) * t.n[2]));
    const float reach = fmaf(h[0], fabsf(t.n[0]), fmaf(h[1], fabsf(t.n[1]), h[2] * fabsf(t.n[2])));
    const float size = scale + fabsf(t.C[0]) + fabsf(t.C[1]) + fabsf(t.C[2]);
    const float margin =
        (size + 1e-38f) * (4e-6f * (fabsf(t.n[0]) + fabsf(t.n[1]) + fabsf(t.n[2])) + 1.5e-12f * ext * ext + 1e-44f) +
        1e-44f;
    return meets && !(fabsf(s) > reach + margin && fabsf(s) < __builtin_inff());
}

// The surface's leaves that meet the box, listed as near: groups of 64 leaves by
// their boxes, a lane each, then the leaves of those that meet it, the next group's
// loaded ahead.  Two dependent loads instead of the patch tree's one a level, which
// is what a query without caps waits for (us, tree / leaf boxes: 10,007 points one
// by one 64 / 52, 6M lattice points 816 / 737, 24 instances 1103 / 1027).  False
// when there are more than the list holds.
__device__ __forceinline__ bool near_leaves(const LeafBox *__restrict__ leaf, int n_leaves, const float (&lo)[3],
                                            const float (&hi)[3], Lists &L, int &n_near) {
    const int lane = lane_id(), n_groups = (n_leaves + kLeafGroup - 1) / kLeafGroup;
    const auto load = [&](int64_t i, bool there, float4 &a, float4 &b) {
        const float4 *q = (const float4 *)(leaf + (there ? i : 0));
        a = q[0];
        b = q[1];
    };
    const auto meets = [&](bool there, const float4 &a, const float4 &b) {
        return there && lo[0] <= b.x && hi[0] >= a.x && lo[1] <= b.y && hi[1] >= a.y && lo[2] <= b.z && hi[2] >= a.z;
    };
    n_near = 0;
    for (int g0 = 0; g0 < n_groups; g0 += 64) {
        float4 a, b;
        load(n_leaves + g0 + lane, g0 + lane < n_groups, a, b);
        uint64_t m = ballot(meets(g0 + lane < n_groups, a, b));
        if (m == 0) continue;
        int i = (g0 + __builtin_ctzll(m)) * kLeafGroup + lane;
        load(i, i < n_leaves, a, b);
        while (m) {
            m &= m - 1;
            const float4 la = a, lb = b;
            const bool there = i < n_leaves;
            if (m) {
                i = (g0 + __builtin_ctzll(m)) * kLeafGroup + lane;
                load(i, i < n_leaves, a, b);
            }
            const bool hit = meets(there, la, lb);
            const uint64_t mn = ballot(hit);
            if (n_near + __popcll(mn) > kNearCap) return false;
            if (hit) L.near[n_near + lanes_below(mn)] = make_uint2(__float_as_uint(la.w), __float_as_uint(lb.w));
            n_near += __popcll(mn);
        }
    }
    wave_sync();
    return true;
}

// The surface's triangles that may meet the box, listed in L.tri from `at` on, at
// most `cap`: their number, -1 if there are more (the surface then keeps to the
// triangles unlisted; with cap 0, 0 is a proof that it does not enter the box).
__device__ __forceinline__ int triangles_near(const LeafBox *__restrict__ leaf, int n_leaves,
                                              const TriRec *__restrict__ rec,
                                              const float (&lo)[3], const float (&hi)[3], Lists &L, int at,
                                              int cap) {
    int n_near, n = 0;
    if (!near_leaves(leaf, n_leaves, lo, hi, L, n_near)) {
        wave_sync();
        return -1;
    }
    const int lane = lane_id();
    float c[3], h[3], scale;
    box_terms(lo, hi, c, h, scale);
    // a leaf a round (a leaf has at most 64 triangles), the next one's loaded ahead
    Tri t;
    uint32_t r = 0;
    bool have = false;
    auto fetch = [&](int i) {
        const uint2 g = L.near[i < n_near ? i : 0];
        have = i < n_near && (uint32_t)lane < g.y;
        r = have ? g.x + (uint32_t)lane : 0u;
        t = load_tri(rec, r);
    };
    if (n_near > 0) fetch(0);
    for (int i = 0; i < n_near; ++i) {
        const bool meets = have && may_meet(t, lo, hi, c, h, scale);
        const uint32_t now = r;
        fetch(i + 1);
        const uint64_t m = ballot(meets);
        if (n + __popcll(m) > cap) {
            n = -1;
            break;
        }
        if (meets) L.tri[at + n + lanes_below(m)] = now;
        n += __popcll(m);
    }
    wave_sync();
    return n;
}

// Change of the winding number from q to each lane's point q + d (d as
// computed; D bounds its length) through the n triangles listed first.
template <typename T>
__device__ __forceinline__ void near_crossings(const TriRec *__restrict__ rec, const Lists &L, int n,
                                               const float (&q)[3], const T (&d)[3], T D, int &delta,
                                               bool &uncertain) {
    const int lane = lane_id();
    for (int i = 0; i < n; i += 64) {
        const int m = min(n - i, 64);
        const Crossing<T> own = make_crossing<T>(load_tri(rec, L.tri[i + (lane < m ? lane : 0)]), q, D);
        for (int j = 0; j < m; ++j) cross(own.from(j), d, delta, uncertain);
    }
}

// Winding number at q, in the surface's box, from the crossings of a ray: 0 at
// its end outside the box, which is reached along one of the axes (the nearest
// face's for turn 0, the others for 1 and 2).  The ray leans by a percent, off
// the planes of regular meshes and thin enough to meet few triangles.  One lane
// per triangle, in double (a float's bound would leave a tenth of the rays
// uncertain).  False if it is not certain.
__device__ __forceinline__ bool ray_winding(const LeafBox *__restrict__ leaf, const TriRec *__restrict__ rec,
                                            const SurfaceDev &sd, const float (&q)[3], int turn, Lists &L,
                                            int &v) {
    int axis = 0;
    float best = __builtin_inff(), to[3];
    for (int c = 0; c < 3; ++c) {
        const float up = sd.hi[c] - q[c], down = q[c] - sd.lo[c], pad = 0.01f * (sd.hi[c] - sd.lo[c]);
        to[c] = up <= down ? sd.hi[c] + pad : sd.lo[c] - pad;
        if (fminf(up, down) < best) {
            best = fminf(up, down);
            axis = c;
        }
    }
    axis = axis + turn >= 3 ? axis + turn - 3 : axis + turn;
    const float len = fabsf(axis == 0 ? to[0] - q[0] : axis == 1 ? to[1] - q[1] : to[2] - q[2]);
    float e[3], lo[3], hi[3];
    double d[3], d2 = 0.0;
    for (int c = 0; c < 3; ++c) {
        const float lean = c == 0 ? 0.0113f : c == 1 ? -0.0071f : 0.0093f;
        e[c] = axis == c ? to[c] : fmaf(len, lean, q[c]);
        lo[c] = fminf(e[c], q[c]);
        hi[c] = fmaxf(e[c], q[c]);
        d[c] = (double)e[c] - (double)q[c];
        d2 += d[c] * d[c];
    }
    const int n = triangles_near(leaf, sd.n_leaves, rec, lo, hi, L, kNearTri, kRayTri);
    int delta = 0;
    bool uncertain = n < 0;
    for (int i = 0; i < n; i += 64) {
        if (lane_id() < n - i) {
            const Tri t = load_tri(rec, L.tri[kNearTri + i + lane_id()]);
            cross(make_crossing<double>(t, q, sqrt(d2) * 1.00001), d, delta, uncertain);
        }
    }
    v = -(int)wave_add((unsigned)delta);
    return ballot(uncertain) == 0;
}

}  // namespace patch
}  // namespace sal

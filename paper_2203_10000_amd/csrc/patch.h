// Device side of the patch tree: which patches of a surface are near a box,
// and the winding sum of one point by a whole wavefront.
#pragma once

#include <hip/hip_runtime.h>

#include "mixed_term.h"
#include "sal_internal.h"
#include "wave.h"

namespace sal {
namespace patch {

constexpr int kNearCap = 96;    // near leaves of one box (96 x ~45 triangles)
constexpr int kFarCap = 384;    // far patches: 3 siblings per level and near node
constexpr int kFrontCap = 64;   // near nodes of one level

// One wavefront's working lists in LDS (4.4 KB: 37 wavefronts fit a CU's LDS,
// so they do not limit occupancy).  Entries are record ranges {begin, count}.
struct Lists {
    uint2 near[kNearCap];
    uint2 far[kFarCap];
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

// The triangle that ends at record r of a strip range starting at `begin`
// (its vertices are that of r and the two before it); false for a head.
struct Tri {
    float X[3], Y[3], Z[3], n[3], len, lim;
};
__device__ __forceinline__ bool load_tri(const Rec32 *__restrict__ rec, uint32_t begin, uint32_t r, Tri &t) {
    const float4 *q = (const float4 *)(rec + r);
    const float4 a = q[0], b = q[1];
    if (b.w == 0.0f) return false;
    const float4 *p1 = (const float4 *)(rec + (r - 1));
    const float4 c = p1[0], d = p1[1];
    t.Z[0] = a.x; t.Z[1] = a.y; t.Z[2] = a.z;
    t.n[0] = a.w; t.n[1] = b.x; t.n[2] = b.y;
    t.len = b.z;
    t.lim = b.w;
    if (d.w == 0.0f) {   // first triangle of a strip: both vertices in the head
        t.X[0] = c.x; t.X[1] = c.y; t.X[2] = c.z;
        t.Y[0] = c.w; t.Y[1] = d.x; t.Y[2] = d.y;
    } else {
        t.Y[0] = c.x; t.Y[1] = c.y; t.Y[2] = c.z;
        const float4 *p2 = (const float4 *)(rec + (r - 2 > begin ? r - 2 : begin));
        const float4 e = p2[0], f = p2[1];
        const bool head = f.w == 0.0f;
        t.X[0] = head ? e.w : e.x;
        t.X[1] = head ? f.x : e.y;
        t.X[2] = head ? f.y : e.z;
    }
    return true;
}

struct PointSum {
    double half;       // sum of atan2(N, D): half the solid angle
    bool on;           // the point lies on a triangle
    bool uncertain;    // some float32 term is not certified (kFloat only)
    unsigned exact;    // exact-sign evaluations, this lane's
    unsigned n_f64;    // float32 terms recomputed in double, this lane's
};

// How a point's terms are evaluated: in float32 (uncertified ones counted),
// in float32 with the uncertified ones in double, or all in double.
enum Mode { kFloat, kMixed, kDouble };

// Half the solid angle of the listed ranges at one point (the same in every
// lane).  Eight groups of eight lanes take ranges in turn, a group the next one
// as it becomes free (all lanes run in step, so the assignment, and with it
// the result, depends on the lists alone); a lane evaluates the triangle that
// ends at its record.  Caps average 25-30 triangles, so wider groups would
// leave more lanes idle at a range's end.
template <Mode MODE>
__device__ __forceinline__ PointSum point_sum(const Rec32 *__restrict__ rec32, const Rec64 *__restrict__ rec64,
                                              const Lists &L, int n_near, int n_far, float px, float py,
                                              float pz, float kap) {
    const int lane = lane_id(), sub = lane & 7;
    const float branch_cut = mixed::kPiF - 0.25f * kap;
    const int items = n_near + n_far;
    const uint64_t leaders = 0x0101010101010101ull;
    PointSum out{0.0, false, false, 0u, 0u};
    float accf = 0.0f;
    double acc = 0.0;
    int next = 0, on = 0;
    uint32_t begin = 0, cur = 0, end = 0;
    bool more = true;
    for (;;) {
        // groups whose range is finished take the next ones in group order
        bool need = more && cur >= end;
        uint64_t m = ballot(need);
        if (m != 0) {
            const int it = next + __popcll(m & leaders & ((1ull << (lane & ~7)) - 1ull));
            if (need) {
                more = it < items;
                if (more) {
                    const uint2 g = it < n_near ? L.near[it] : L.far[it - n_near];
                    begin = g.x;
                    cur = g.x;
                    end = g.x + g.y;
                }
            }
            next += __popcll(m & leaders);
        }
        if (ballot(more) == 0) break;
        const uint32_t r = cur + (uint32_t)sub;
        Tri t;
        if (more && r < end && load_tri(rec32, begin, r, t)) {
            if (MODE == kDouble) {
                const mixed::F64Term d = mixed::f64_triangle(t.X[0], t.X[1], t.X[2], t.Y[0], t.Y[1], t.Y[2],
                                                             rec64[r].v, px, py, pz);
                acc += d.half;
                on |= d.on;
                out.exact += d.exact;
            } else {
                const float ax = t.X[0] - px, ay = t.X[1] - py, az = t.X[2] - pz;
                const float bx = t.Y[0] - px, by = t.Y[1] - py, bz = t.Y[2] - pz;
                const float cx = t.Z[0] - px, cy = t.Z[1] - py, cz = t.Z[2] - pz;
                const float ar = __builtin_amdgcn_sqrtf(fmaf(ax, ax, fmaf(ay, ay, az * az)));
                const float br = __builtin_amdgcn_sqrtf(fmaf(bx, bx, fmaf(by, by, bz * bz)));
                const float cr = __builtin_amdgcn_sqrtf(fmaf(cx, cx, fmaf(cy, cy, cz * cz)));
                const float e01 = fmaf(ax, bx, fmaf(ay, by, az * bz));
                const float e02 = fmaf(ax, cx, fmaf(ay, cy, az * cz));
                const float e12 = fmaf(bx, cx, fmaf(by, cy, bz * cz));
                const float nn = fmaf(cx, t.n[0], fmaf(cy, t.n[1], cz * t.n[2]));   // 32 N
                const float mm = ar * br * cr;
                const float dd = fmaf(e12, ar, fmaf(e02, br, fmaf(e01, cr, mm)));
                const float lim = fmaf(t.lim, cr, fmaf(kap, mm, fabsf(nn)));
                if (__builtin_expect(dd > lim, 1)) {   // |N / D| < 1/32: the series
                    const float u = nn * __builtin_amdgcn_rcpf(dd);
                    const float s2 = u * u;
                    accf = fmaf(u, fmaf(fmaf(mixed::kA2, s2, mixed::kA1), s2, mixed::kA0), accf);
                } else {
                    const float n1 = nn * (1.0f / kNScale);
                    const float ang = atan2f(n1, dd);
                    const float thr = fmaf(cr, kap * t.len, kap * mm);
                    const bool ill = !(fmaxf(fabsf(n1), fabsf(dd)) > thr) || fabsf(ang) > branch_cut;
                    if (!ill) {
                        accf += ang;
                    } else if (MODE == kFloat) {
                        out.uncertain = true;
                    } else {
                        const mixed::F64Term d = mixed::f64_triangle(t.X[0], t.X[1], t.X[2], t.Y[0], t.Y[1],
                                                                     t.Y[2], rec64[r].v, px, py, pz);
                        acc += d.half;
                        on |= d.on;
                        out.exact += d.exact;
                        out.n_f64 += 1u;
                    }
                }
            }
        }
        cur += 8;
    }
    acc += (double)accf;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) acc += __shfl_xor(acc, d);
    out.half = acc;
    out.on = ballot(on != 0) != 0;
    out.uncertain = ballot(out.uncertain) != 0;
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
// the double rounding of n; twice that is taken.  A lane whose sign is within a
// bound, and not settled by the others, is uncertain.
template <typename T>
struct Bounds;
template <>
struct Bounds<float> {
    static constexpr float edge = 24.0f * 5.9604645e-8f, plane = 20.0f * 5.9604645e-8f;
    static constexpr float normal = 1.5e-13f;   // 32 (scaled normals) x 4.7e-15, per L^2
    static constexpr float huge = 1e37f;
};
template <>
struct Bounds<double> {
    static constexpr double edge = 24.0 * 1.1102230246251565e-16, plane = 20.0 * 1.1102230246251565e-16;
    static constexpr double normal = 5e-15;
    static constexpr double huge = 1e300;
};

// What 64 points need of one triangle, relative to q.
template <typename T>
struct Crossing {
    T e[3][3];   // edge products (X - q) x (Y - q) and on
    T n[3], s;   // side * normal, side * n . (Z - q)
    T tol_e, tol_s;
    int side;    // +1: q outside (n . (q - Z) > 0), -1: inside, 0: not certain

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
__device__ __forceinline__ Crossing<T> make_crossing(const Tri &t, const T (&n)[3], const float (&q)[3], T D) {
    typedef Bounds<T> B;
    Crossing<T> o;
    T v[3][3], l2 = 0;
    for (int c = 0; c < 3; ++c) {
        v[0][c] = (T)t.X[c] - (T)q[c];
        v[1][c] = (T)t.Y[c] - (T)q[c];
        v[2][c] = (T)t.Z[c] - (T)q[c];
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
    o.tol_e = B::edge * l2 * D;
    o.tol_s = reach * (B::plane * len + B::normal * l2);
    // far out of range: nothing is certain (also catches NaN)
    if (!(l2 * reach < B::huge) || !(len * reach < B::huge)) o.tol_e = o.tol_s = B::huge;
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

// Whether triangle t may meet the box of centre c and half extents h (scale: |c|
// + h): its own box does (exact comparisons) and its plane passes within the
// box's radius, with a margin some thirty times the products' rounding.
__device__ __forceinline__ bool may_meet(const Tri &t, const float (&lo)[3], const float (&hi)[3],
                                         const float (&c)[3], const float (&h)[3], float scale) {
    bool meets = true;
    float ext = 0.0f;
    for (int k = 0; k < 3; ++k) {
        const float a = fminf(fminf(t.X[k], t.Y[k]), t.Z[k]), b = fmaxf(fmaxf(t.X[k], t.Y[k]), t.Z[k]);
        meets = meets && a <= hi[k] && b >= lo[k];
        ext = fmaxf(ext, b - a);
    }
    const float s = fmaf(c[0] - t.Z[0], t.n[0], fmaf(c[1] - t.Z[1], t.n[1], (c[2] - t.Z[2]) * t.n[2]));
    const float reach = fmaf(h[0], fabsf(t.n[0]), fmaf(h[1], fabsf(t.n[1]), h[2] * fabsf(t.n[2])));
    const float size = scale + fabsf(t.Z[0]) + fabsf(t.Z[1]) + fabsf(t.Z[2]);
    const float margin = size * (4e-6f * (fabsf(t.n[0]) + fabsf(t.n[1]) + fabsf(t.n[2])) + 1.5e-12f * ext * ext);
    return meets && !(fabsf(s) > reach + margin);
}

// Change of the winding number from q to each lane's point q + d (d as
// computed; D bounds its length) through the near list's triangles.
template <typename T>
__device__ __forceinline__ void near_crossings(const Rec32 *__restrict__ rec32, const Rec64 *__restrict__ rec64,
                                               const Lists &L, int n_near, const float (&lo)[3],
                                               const float (&hi)[3], const float (&q)[3], const T (&d)[3], T D,
                                               int &delta, bool &uncertain) {
    const int lane = lane_id();
    float c[3], h[3];
    for (int k = 0; k < 3; ++k) {
        c[k] = 0.5f * lo[k] + 0.5f * hi[k];
        h[k] = 0.5f * hi[k] - 0.5f * lo[k];
    }
    const float scale = fabsf(c[0]) + fabsf(c[1]) + fabsf(c[2]) + h[0] + h[1] + h[2];
    for (int i = 0; i < n_near; ++i) {
        const uint2 g = L.near[i];
        const uint32_t begin = (uint32_t)__builtin_amdgcn_readfirstlane((int)g.x);
        const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)g.y);
        for (uint32_t o = 0; o < n; o += 64) {
            const uint32_t r = begin + o + (uint32_t)lane;
            Tri t;
            bool meets = false;
            if (o + lane < n && load_tri(rec32, begin, r, t)) meets = may_meet(t, lo, hi, c, h, scale);
            uint64_t m = ballot(meets);
            if (m == 0) continue;
            Crossing<T> own;
            if (meets) {
                T nn[3];
                for (int k = 0; k < 3; ++k) nn[k] = sizeof(T) == 8 ? (T)rec64[r].v[3 + k] : (T)t.n[k];
                own = make_crossing<T>(t, nn, q, D);
            }
            for (; m; m &= m - 1) cross(own.from(__builtin_ctzll(m)), d, delta, uncertain);
        }
    }
}

}  // namespace patch
}  // namespace sal

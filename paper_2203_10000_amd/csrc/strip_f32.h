// Float32 strip walk: 64 points, one per lane, against the same strips.
#pragma once

#include <hip/hip_runtime.h>

#include "sal_internal.h"

namespace sal {
namespace f32 {

constexpr double kInv2Pi = 0.15915494309189533577;
constexpr float kPiF = 3.14159265358979323846f;

// atan(t) for |t| <= 1/32 given u = 32 t (the record normals carry the
// factor 32):  u (1/32 - u^2 / (3 32^3)), the Taylor series to t^3; the first
// omitted term, t^5 / 5, is below 2e-7 t.
constexpr float kA0 = 0.03125f;
constexpr float kA1 = -1.0172526042e-05f;   // -1 / (3 * 32768)
static_assert(kNScale == 32.0f, "series constants assume normals scaled by 32");

__device__ __forceinline__ uint64_t ballot(bool b) { return __builtin_amdgcn_ballot_w64(b); }

__device__ __forceinline__ int lane_id() {
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// Number of set bits of m below this lane.
__device__ __forceinline__ int lanes_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ int64_t bcast_i64(int64_t v, int src) {
    const int lo = __builtin_amdgcn_readlane((int)(uint32_t)v, src);
    const int hi = __builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), src);
    return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

__device__ __forceinline__ bool finite3(float x, float y, float z) {
    return __builtin_isfinite(x) && __builtin_isfinite(y) && __builtin_isfinite(z);
}

// ------------------------------------------------------------------ float32
// Records are read through the constant address space: the address is the
// same for every lane, so each record is one scalar load into SGPRs.
typedef __attribute__((address_space(4))) const Rec32 CRec32;
typedef __attribute__((address_space(4))) const Rec64 CRec64;
typedef __attribute__((address_space(4))) const SurfaceDev CSurf;

struct Vtx {
    float x, y, z, r;   // vertex - p and its length
};

// The eight floats of one triangle record, held in SGPRs.
struct TriRec {
    float v[8];
};

// The load is volatile only to pin it where the source puts it: the compiler
// would otherwise sink a prefetch down to the end of the loop body, next to
// the copy that consumes it.  It is still one scalar load.
__device__ __forceinline__ TriRec load_rec(const CRec32 *p) {
    typedef float F8 __attribute__((ext_vector_type(8)));
    typedef __attribute__((address_space(4))) const volatile F8 VF8;
    const F8 w = *(const VF8 *)p;
    TriRec r;
#pragma unroll
    for (int c = 0; c < 8; ++c) r.v[c] = w[c];
    return r;
}

// One strip step: the triangle (O, N, Z) with Z and its normal in record `rec`.
// Z is written to the free slot F; the caller rotates the three slots (O, N, F)
// -> (N, F, O) instead of moving registers.
__device__ __forceinline__ void f32_step(const Vtx &O, const Vtx &N, Vtx &F, float &e01, float &rr01,
                                         float &acc, float &accn, const TriRec &rec, float px,
                                         float py, float pz, uint64_t good_mask, float kap,
                                         float branch_cut, uint64_t &cmask) {
    const float x2 = rec.v[0] - px, y2 = rec.v[1] - py, z2 = rec.v[2] - pz;
    const float r2 = __builtin_amdgcn_sqrtf(fmaf(x2, x2, fmaf(y2, y2, z2 * z2)));
    const float e02 = fmaf(O.x, x2, fmaf(O.y, y2, O.z * z2));
    const float e12 = fmaf(N.x, x2, fmaf(N.y, y2, N.z * z2));
    const float nn = fmaf(x2, rec.v[3], fmaf(y2, rec.v[4], z2 * rec.v[5]));   // 32 N
    const float mm = rr01 * r2;                                               // |a||b||c|
    const float dd = fmaf(e12, O.r, fmaf(e02, N.r, fmaf(e01, r2, mm)));
    // small-angle path: |N/D| < 1/32, D > kappa |a||b||c|, D > 5 |n| |c|
    const float lim = fmaf(rec.v[7], r2, fmaf(kap, mm, fabsf(nn)));
    const uint64_t near = ballot(!(dd > lim)) & good_mask;
    // The hint lays the series out as the fall-through path (without it the
    // atan2 block fell through and the common path took three branches per
    // step: 2 % of a launch over 82k triangles).
    if (__builtin_expect(near == 0, 1)) {
        const float u = nn * __builtin_amdgcn_rcpf(dd);
        acc = fmaf(u, fmaf(kA1, u * u, kA0), acc);
    } else {
        const float n1 = nn * (1.0f / kNScale);
        const float ang = atan2f(n1, dd);
        const float thr = fmaf(r2, kap * rec.v[6], kap * mm);
        const bool ill = !(fmaxf(fabsf(n1), fabsf(dd)) > thr);   // (NaN is ill)
        const bool cut = fabsf(ang) > branch_cut;
        cmask |= (ballot(ill) | ballot(cut)) & good_mask;
        accn += ang;
    }
    rr01 = N.r * r2;
    e01 = e12;
    F.x = x2;
    F.y = y2;
    F.z = z2;
    F.r = r2;
}

// Sums atan2(N, D) = Omega / 2 over the strips in records [rec_begin,
// rec_end) for this lane's point: S += per-strip float32 sums, cmask |= lanes
// whose pair is ill-conditioned.
__device__ __forceinline__ void strips_sum(const CRec32 *rec, int64_t rec_begin, int64_t rec_end,
                                           float px, float py, float pz, uint64_t good_mask, float kap,
                                           float branch_cut, double &S, uint64_t &cmask) {
    for (int64_t r = rec_begin; r < rec_end;) {
        const CRec32 *h = rec + r;
        const int m = __float_as_int(h->v[6]);
        Vtx A, B, C;
        // Small-angle terms and full-atan2 terms go to separate float sums,
        // so the two paths do not merge one register (no copy per step).
        float acc = 0.0f, accn = 0.0f;
        A.x = h->v[0] - px; A.y = h->v[1] - py; A.z = h->v[2] - pz;
        B.x = h->v[3] - px; B.y = h->v[4] - py; B.z = h->v[5] - pz;
        A.r = __builtin_amdgcn_sqrtf(fmaf(A.x, A.x, fmaf(A.y, A.y, A.z * A.z)));
        B.r = __builtin_amdgcn_sqrtf(fmaf(B.x, B.x, fmaf(B.y, B.y, B.z * B.z)));
        float e01 = fmaf(A.x, B.x, fmaf(A.y, B.y, A.z * B.z));
        float rr01 = A.r * B.r;
        // Triangle records are prefetched one step ahead: each step first
        // waits for the scalar loads in flight (the record it is about to
        // use), then issues the load of the next record, then computes, so a
        // load overlaps a whole step.  The explicit wait orders the two
        // (scalar loads can return out of order, so any wait is a wait for
        // all of them).  Indices are clamped to the strip's last record.
        const CRec32 *tr = h + 1;
        const int last = m - 1;
        TriRec c0 = load_rec(tr), c1, c2;
        int t = 0;
        for (; t + 2 < m; t += 3) {
            __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
            c1 = load_rec(tr + (t + 1));
            __builtin_amdgcn_sched_barrier(0);     // keep the step's arithmetic below
            f32_step(A, B, C, e01, rr01, acc, accn, c0, px, py, pz, good_mask, kap, branch_cut, cmask);
            __builtin_amdgcn_s_waitcnt(0xc07f);
            c2 = load_rec(tr + (t + 2));
            __builtin_amdgcn_sched_barrier(0);
            f32_step(B, C, A, e01, rr01, acc, accn, c1, px, py, pz, good_mask, kap, branch_cut, cmask);
            __builtin_amdgcn_s_waitcnt(0xc07f);
            c0 = load_rec(tr + (t + 3 < last ? t + 3 : last));
            __builtin_amdgcn_sched_barrier(0);
            f32_step(C, A, B, e01, rr01, acc, accn, c2, px, py, pz, good_mask, kap, branch_cut, cmask);
        }
        __builtin_amdgcn_s_waitcnt(0xc07f);
        if (t < m) {
            f32_step(A, B, C, e01, rr01, acc, accn, c0, px, py, pz, good_mask, kap, branch_cut, cmask);
            if (t + 1 < m) {
                c1 = load_rec(tr + (t + 1));
                f32_step(B, C, A, e01, rr01, acc, accn, c1, px, py, pz, good_mask, kap, branch_cut, cmask);
            }
        }
        S += (double)acc + (double)accn;
        r += m + 1;
    }
}

}  // namespace f32
}  // namespace sal

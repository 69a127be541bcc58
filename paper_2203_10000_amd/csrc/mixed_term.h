// Mixed-precision terms of a recomputed pair: the winding number of a closed
// surface is an integer away from the surface (section 2.1.3 labels by it), so
// a (point, surface) pair only needs every triangle term correct to far less
// than 1/2 in total.  A term that float32 certifies (the small-angle test of
// the pair loop, or the full atan2 without its conditioning flags) is kept in
// float32; the others are recomputed in double with the exact-sign guard.  The
// float32 terms are the ones the pair loop accepts for unflagged pairs.
#pragma once

#include <hip/hip_runtime.h>

#include "sal_internal.h"
#include "vos_f64.h"

namespace sal {
namespace mixed {

constexpr float kPiF = 3.14159265358979323846f;
// atan(t) = u (1/32 - u^2 / (3 32^3) + u^4 / (5 32^5)) for u = 32 t,
// |t| <= 1/32: the pair loop's small-angle range, with one more term of the
// series (first omitted term below 1e-10 t).
constexpr float kA0 = 0.03125f;
constexpr float kA1 = -1.0172526042e-05f;   // -1 / (3 * 32768)
constexpr float kA2 = 5.9604644775e-09f;    //  1 / (5 * 33554432)
static_assert(kNScale == 32.0f, "series constants assume normals scaled by 32");

struct F64Term {
    double half;      // atan2(N, D)
    int on;           // the point lies on the closed triangle
    unsigned exact;   // exact-sign evaluations made
};

// One triangle (X, Y, Z) in double with the exact-sign guard; Z and the
// double normal come from its FP64 record.  Out of line and by value: it is
// rare, and inlined its registers would count against the float32 walk.
__device__ __noinline__ F64Term f64_triangle(float x0, float x1, float x2, float y0, float y1,
                                             float y2, const double *rec, float px, float py,
                                             float pz) {
    const double Xd[3] = {x0, x1, x2}, Yd[3] = {y0, y1, y2};
    const double pd[3] = {px, py, pz};
    const float pf[3] = {px, py, pz};
    StripF64 st;
    f64_strip_window(st, Xd, Yd, pd);
    F64Term r{0.0, 0, 0u};
    r.half = f64_strip_tri(st, rec, pd, pf, &r.on, &r.exact);
    return r;
}

}  // namespace mixed
}  // namespace sal

// Van Oosterom-Strackee solid angle of one triangle in double precision (the
// FP64 form, and the terms float32 does not certify).
//
// For a point p and triangle (A, B, C) with a = A - p, b = B - p, c = C - p:
//   Omega / 2 = atan2(N, D),  N = a . (b x c) = c . n,  n = (B - A) x (C - A),
//   D = |a||b||c| + (a.b)|c| + (a.c)|b| + (b.c)|a|
// (Van Oosterom & Strackee, IEEE Trans. Biomed. Eng. 30(2), 1983; the
// paper's section 2.1.3 labels a point by the solid angle of a closed surface
// over 4 pi).
//
// When |N| is below its rounding-error bound the sign comes from the exact
// predicate; a point exactly on the triangle's plane and inside the closed
// triangle is "on the surface" (enclosed), otherwise it contributes 0.  Cap
// triangles take the computed sign: the point is never near one, so where the
// sign is uncertain the angle is as small as its rounding.
//
// The winding number of a closed surface is an integer away from the surface, so
// in the float32 form a (point, surface) pair only needs every term correct to
// far less than 1/2 in total: a term that float32 certifies (the small-angle
// test, or the full atan2 without its conditioning flags) stays in float32, the
// others come here.
#pragma once

#include <hip/hip_runtime.h>

#include "exact_dev.h"
#include "sal_internal.h"

namespace sal {

constexpr float kPiF = 3.14159265358979323846f;
// atan(t) = u (1/32 - u^2 / (3 32^3) + u^4 / (5 32^5)) for u = 32 t,
// |t| <= 1/32 (first omitted term below 1e-10 t).
constexpr float kA0 = 0.03125f;
constexpr float kA1 = -1.0172526042e-05f;   // -1 / (3 * 32768)
constexpr float kA2 = 5.9604644775e-09f;    //  1 / (5 * 33554432)
static_assert(kNScale == 32.0f, "series constants assume normals scaled by 32");

struct Tri {
    float A[3], B[3], C[3], n[3];   // n scaled by kNScale
};

struct F64Term {
    double half;      // atan2(N, D)
    int on;           // the point lies on the closed triangle
    unsigned exact;   // exact-sign evaluations made
};

// Out of line and by value: inlined, its registers would count against the
// loops around it.
__device__ __noinline__ F64Term f64_term(const Tri t, float px, float py, float pz, bool cap) {
    const double p[3] = {px, py, pz};
    double a[3], b[3], c[3], e1[3], e2[3];
    for (int k = 0; k < 3; ++k) {
        a[k] = (double)t.A[k] - p[k];
        b[k] = (double)t.B[k] - p[k];
        c[k] = (double)t.C[k] - p[k];
        e1[k] = (double)t.B[k] - (double)t.A[k];
        e2[k] = (double)t.C[k] - (double)t.A[k];
    }
    const double ra = sqrt(a[0] * a[0] + a[1] * a[1] + a[2] * a[2]);
    const double rb = sqrt(b[0] * b[0] + b[1] * b[1] + b[2] * b[2]);
    const double rc = sqrt(c[0] * c[0] + c[1] * c[1] + c[2] * c[2]);
    const double ab = a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
    const double ac = a[0] * c[0] + a[1] * c[1] + a[2] * c[2];
    const double bc = b[0] * c[0] + b[1] * c[1] + b[2] * c[2];
    const double n[3] = {e1[1] * e2[2] - e1[2] * e2[1], e1[2] * e2[0] - e1[0] * e2[2],
                         e1[0] * e2[1] - e1[1] * e2[0]};
    double num = c[0] * n[0] + c[1] * n[1] + c[2] * n[2];
    const double den = ra * rb * rc + ab * rc + ac * rb + bc * ra;
    F64Term r{0.0, 0, 0u};
    if (!cap) {
        const double q1 = e1[0] * e1[0] + e1[1] * e1[1] + e1[2] * e1[2];
        const double q2 = e2[0] * e2[0] + e2[1] * e2[1] + e2[2] * e2[2];
        if (fabs(num) <= kGuardEps * rc * sqrt(q1 * q2)) {
            r.exact = 1u;
            const float P[3] = {px, py, pz};
            const int o = exact_orient3d(P, t.A, t.B, t.C);
            if (o == 0) {
                r.on = exact_in_triangle(P, t.A, t.B, t.C) ? 1 : 0;
                return r;
            }
            const double mag = num != 0.0 ? fabs(num) : 2.2250738585072014e-308;
            num = o > 0 ? mag : -mag;
            r.half = atan2(num, den);
            return r;
        }
    }
    if (den > 16.0 * fabs(num)) {
        // |N / D| < 1/16 with D > 0: atan2(N, D) = atan(t), t = N / D, by its
        // Taylor series to t^13 (the first omitted term is below 1e-18 t)
        const double x = num / den, q = x * x;
        double poly = 1.0 / 13.0;
        poly = fma(poly, q, -1.0 / 11.0);
        poly = fma(poly, q, 1.0 / 9.0);
        poly = fma(poly, q, -1.0 / 7.0);
        poly = fma(poly, q, 1.0 / 5.0);
        poly = fma(poly, q, -1.0 / 3.0);
        r.half = fma(x * q, poly, x);
    } else {
        r.half = atan2(num, den);
    }
    return r;
}

}  // namespace sal

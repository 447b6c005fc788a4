// Device functions of the surface integrals (gfx950): complex helpers, the rational
// Bezier element maps, the local B-splines and the pulled-back kernels.
// All floating point is fp64; complex values are double2 (re, im).
#pragma once

#include <hip/hip_runtime.h>

#include "common.h"

namespace igb {

// --------------------------------------------------------------------------
// small device helpers
// --------------------------------------------------------------------------
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// c + a * b
__device__ __forceinline__ double2 cfma(double2 a, double2 b, double2 c) {
    return make_double2(fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y)));
}
__device__ __forceinline__ double2 cscale(double2 a, double s) { return make_double2(a.x * s, a.y * s); }

// Bernstein polynomials of degree p <= 3 on [0,1] and their derivatives
__device__ __forceinline__ void bernstein(int p, double s, double* b, double* db) {
    const double t = 1.0 - s;
    if (p == 0) {
        b[0] = 1; db[0] = 0;
    } else if (p == 1) {
        b[0] = t; b[1] = s; db[0] = -1; db[1] = 1;
    } else if (p == 2) {
        b[0] = t * t; b[1] = 2 * s * t; b[2] = s * s;
        db[0] = -2 * t; db[1] = 2 * (t - s); db[2] = 2 * s;
    } else {
        b[0] = t * t * t; b[1] = 3 * s * t * t; b[2] = 3 * s * s * t; b[3] = s * s * s;
        db[0] = -3 * t * t; db[1] = 3 * t * t - 6 * s * t; db[2] = 6 * s * t - 3 * s * s; db[3] = 3 * s * s;
    }
}

struct GeoPt {
    double x[3];   // F
    double fs[3];  // dF/ds (element-local)
    double ft[3];  // dF/dt
};

// rational Bezier element map at local (s, t)
__device__ __forceinline__ void eval_geo(const double* __restrict__ bez, int pu, int pv, double s,
                                         double t, GeoPt& g) {
    double bu[4], dbu[4], bv[4], dbv[4];
    bernstein(pu, s, bu, dbu);
    bernstein(pv, t, bv, dbv);
    double P[4] = {0, 0, 0, 0}, Ps[4] = {0, 0, 0, 0}, Pt[4] = {0, 0, 0, 0};
    for (int j = 0; j <= pv; ++j) {
        double rP[4] = {0, 0, 0, 0}, rPs[4] = {0, 0, 0, 0};
        for (int i = 0; i <= pu; ++i) {
            const double* H = bez + (j * (PGMAX + 1) + i) * 4;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                rP[c] = fma(bu[i], H[c], rP[c]);
                rPs[c] = fma(dbu[i], H[c], rPs[c]);
            }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            P[c] = fma(bv[j], rP[c], P[c]);
            Ps[c] = fma(bv[j], rPs[c], Ps[c]);
            Pt[c] = fma(dbv[j], rP[c], Pt[c]);
        }
    }
    const double iw = 1.0 / P[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        g.x[c] = P[c] * iw;
        g.fs[c] = (Ps[c] - g.x[c] * Ps[3]) * iw;
        g.ft[c] = (Pt[c] - g.x[c] * Pt[3]) * iw;
    }
}

__device__ __forceinline__ void cross3(const double* a, const double* b, double* c) {
    c[0] = a[1] * b[2] - a[2] * b[1];
    c[1] = a[2] * b[0] - a[0] * b[2];
    c[2] = a[0] * b[1] - a[1] * b[0];
}

// local B-splines b_{ex+a}(s), a = 0..p, from the element's extraction rows
template <int P>
__device__ __forceinline__ void eval_basis1(const double* __restrict__ C, double s, double* phi, double* dphi) {
    double b[4], db[4];
    bernstein(P, s, b, db);
#pragma unroll
    for (int a = 0; a <= P; ++a) {
        double v = 0, d = 0;
#pragma unroll
        for (int k = 0; k <= P; ++k) {
            v = fma(C[a * (P + 1) + k], b[k], v);
            d = fma(C[a * (P + 1) + k], db[k], d);
        }
        phi[a] = v;
        if (dphi) dphi[a] = d;
    }
}

__device__ __forceinline__ void d4_apply(int code, double s, double t, double& a, double& b) {
    a = s;
    b = t;
    if (code & 4) {
        double x = a;
        a = b;
        b = x;
    }
    if (code & 1) a = 1.0 - a;
    if (code & 2) b = 1.0 - b;
}

struct ElemRef {
    const double* bez;
    int pu, pv, ex, ey;
};

__device__ __forceinline__ ElemRef elem_ref(const double* bez, const int* pg, int nel1, int64_t e) {
    ElemRef r;
    r.bez = bez + e * NBZ * 4;
    r.pu = pg[2 * e];
    r.pv = pg[2 * e + 1];
    int64_t rem = e % (int64_t(nel1) * nel1);
    r.ey = int(rem / nel1);
    r.ex = int(rem % nel1);
    return r;
}

// The pulled-back kernel of the sound-soft family  ck a_y H (x-y).n~_x + cv a_x a_y G
// with G = e^{i kappa r}/(4 pi r), H = G (i kappa r - 1)/r^2 (Sec. 4.2, eq. of
// the pulled-back kernel, applied to K* and V): ck = 1, cv = -i eta for the
// CFIE of the D2N system, cv = 1 (V alone) or ck = 1, cv = 0 (K* alone) for the
// single-layer formulations.
__device__ __forceinline__ double2 kernel_soft(const double* X, const double* NX, double ax,
                                               const double* Y, double ay, double kappa, SoftMix mix) {
    const double d0 = X[0] - Y[0], d1 = X[1] - Y[1], d2 = X[2] - Y[2];
    const double r2 = d0 * d0 + d1 * d1 + d2 * d2;
    const double r = sqrt(r2);
    const double ir = 1.0 / r;
    const double kr = kappa * r;
    double sn, cs;
    sincos(kr, &sn, &cs);
    const double dn = d0 * NX[0] + d1 * NX[1] + d2 * NX[2];
    const double c4 = 0.07957747154594767 * ir;        // 1/(4 pi r)
    const double h = mix.ck * ay * dn * ir * ir * c4;   // ck a_y (x-y).n~_x / (4 pi r^3)
    const double v = ax * ay * c4;
    return make_double2(h * (-cs - sn * kr) + v * (mix.cv.x * cs - mix.cv.y * sn),
                        h * (cs * kr - sn) + v * (mix.cv.x * sn + mix.cv.y * cs));
}

}  // namespace igb

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

// wavefront-wide ordering of LDS traffic inside one wave
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 1/x and 1/sqrt(x) for normal x: the hardware estimates (about 2^-24) and one
// third-order correction; the result is within an ulp or two, at a fraction of
// the instructions of the correctly rounded division and square root.
__device__ __forceinline__ double rcp_fast(double x) {
    const double y = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, y, 1.0);
    return fma(y, fma(e, e, e), y);
}
__device__ __forceinline__ double rsqrt_fast(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double h = fma(-x * y, y, 1.0);
    return fma(y * h, fma(h, 0.375, 0.5), y);
}

// the 32-bit words of a double
struct Words {
    unsigned lo, hi;
};
__host__ __device__ __forceinline__ unsigned low_word(double x) { return __builtin_bit_cast(Words, x).lo; }
__host__ __device__ __forceinline__ unsigned high_word(double x) { return __builtin_bit_cast(Words, x).hi; }
__host__ __device__ __forceinline__ double from_words(unsigned hi, unsigned lo) {
    return __builtin_bit_cast(double, Words{lo, hi});
}

// sin(x) and cos(x) to 2e-16 for |x| < 2^48 and 1e-15 for |x| < 2^50: x reduced by
// the nearest multiple of pi/2 (read off the low bits of x 2/pi + 1.5 2^52) in two
// fused steps with pi/2 = A + B to 107 bits, then polynomials on [-pi/4, pi/4]
// (interpolants of (sin r - r)/r^3 and (cos r - 1 + r^2/2)/r^4 in r^2 at six
// Chebyshev points; truncation below 1.4e-17).  Without the libm function's
// branch for huge arguments: from 2^44 the rounding of 2/pi can pick the
// neighbouring multiple, which leaves |r| a little above pi/4 (up to 0.85 at 2^50);
// from 2^51, where the spacing of doubles approaches a radian, the values are only
// bounded: an |r| above 1 has its high word cleared, which leaves 0 (a comparison and
// one select, the price of two clamps; unlike fmin and fmax they leave a NaN a
// NaN, and NaN and infinite arguments give NaN).  About 35 instructions.
__host__ __device__ __forceinline__ void sincos_fast(double x, double& sn, double& cs) {
    const double MAGIC = 6755399441055744.0;   // 1.5 * 2^52
    const double t = fma(x, 0x1.45f306dc9c883p-1, MAGIC);
    const double n = t - MAGIC;
    double r = fma(n, -0x1.921fb54442d18p+0, x);
    r = fma(n, -0x1.1a62633145c07p-54, r);
    r = from_words(fabs(r) > 1.0 ? 0u : high_word(r), low_word(r));
    const double z = r * r;
    double S = fma(z, 0x1.5e0af186af739p-33, -0x1.ae600a926c89ap-26);
    S = fma(z, S, 0x1.71de37961e4c6p-19);
    S = fma(z, S, -0x1.a01a019e8357dp-13);
    S = fma(z, S, 0x1.1111111110bb1p-7);
    S = fma(z, S, -0x1.5555555555555p-3);
    const double s = fma(r * z, S, r);
    double C = fma(z, -0x1.907d7aebd5e3dp-37, 0x1.1eeb68b109173p-29);
    C = fma(z, C, -0x1.27e4fa17a41b4p-22);
    C = fma(z, C, 0x1.a01a019f4e867p-16);
    C = fma(z, C, -0x1.6c16c16c16966p-10);
    C = fma(z, C, 0x1.5555555555555p-5);
    const double c = fma(z * z, C, fma(z, -0.5, 1.0));
    const unsigned q = low_word(t);
    const double a = (q & 1) ? c : s, b = (q & 1) ? s : c;
    sn = from_words(high_word(a) ^ ((q & 2) << 30), low_word(a));
    cs = from_words(high_word(b) ^ (((q + 1) & 2) << 30), low_word(b));
}

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

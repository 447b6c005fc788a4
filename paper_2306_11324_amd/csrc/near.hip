// Near field of the igafmm library (gfx950): the Galerkin blocks of close and touching
// element pairs by quadrature, gathered into the CSR matrix of the solution space.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "common.h"
#include "quadrature_device.h"

namespace igb {

// --------------------------------------------------------------------------
// Near field: regular element pairs (tensor Gauss of order n on both elements)
// --------------------------------------------------------------------------
constexpr int NEAR_THREADS = 256;

struct NearArgs {
    const double* bez;
    const int* pg;
    const double* C1;
    const double* gl;        // [NGMAX+1][2][NGMAX]: Gauss nodes / weights on [0,1] per order
    const int* pair_e;       // near pair -> target element
    const int* pair_f;       // near pair -> source element
    const int* pair_kind;
    const int* list;         // near pairs handled by this launch
    int64_t nlist;
    int64_t slot0;           // staging slot = pair - slot0
    double2* stage;          // [slots][nloc*nloc]
    int nel1;
    double kappa, eta;       // eta: coupling of the sound-hard CFIE
    SoftMix mix;             // kernel of the sound-soft family
    HardMix hmix;            // kernel of the sound-hard family
    double2 cm;              // multiple of the mass matrix added on identical pairs
    // singular rules: per class (0 vertex, 1 edge, 2 identical) points (s1,s2,r1,r2,w)
    const double* rule[3];
    int rule_n[3];
    int mass_order;
};

// Kernel values at one point pair (element-local coordinates, n~ unnormalised):
//   soft: s = ck a_y H (x-y).n~_x + cv a_x a_y G                      (ck K* + cv V)
//   hard: s = ck a_x H (y-x).n~_y - cw kappa^2 G n~_x.n~_y            (ck K, kappa^2 part of cw W)
//         g = cw G, multiplying the curl product c_i(x).c_j(y)         (curl part of cw W)
//         (the CFIE: ck = -1, cw = -i eta)
struct KVal {
    double2 s, g;
};

template <bool HARD>
__device__ __forceinline__ KVal kernel_pair(const double* X, const double* NX, double ax, const double* Y,
                                            const double* NY, double ay, double kappa, SoftMix mix, HardMix hmix) {
    KVal k;
    if (!HARD) {
        k.s = kernel_soft(X, NX, ax, Y, ay, kappa, mix);
        k.g = make_double2(0, 0);
        return k;
    }
    const double d0 = X[0] - Y[0], d1 = X[1] - Y[1], d2 = X[2] - Y[2];
    const double r = sqrt(d0 * d0 + d1 * d1 + d2 * d2);
    const double ir = 1.0 / r;
    const double kr = kappa * r;
    double sn, cs;
    sincos(kr, &sn, &cs);
    const double c4 = 0.07957747154594767 * ir;
    const double dny = d0 * NY[0] + d1 * NY[1] + d2 * NY[2];
    const double nn = NX[0] * NY[0] + NX[1] * NY[1] + NX[2] * NY[2];
    // K kernel a_x H (y-x).n~_y = kn (cs + i sn) (i kr - 1), kn = -a_x (x-y).n~_y / (4 pi r^3)
    const double kn = -ax * dny * ir * ir * c4;
    const double2 kk = make_double2(kn * (-cs - sn * kr), kn * (cs * kr - sn));
    const double v = -kappa * kappa * nn * c4;   // W's kappa^2 part: v (cs + i sn)
    const double2 w = make_double2(v * cs, v * sn);
    const double2 g = make_double2(c4 * cs, c4 * sn);
    k.s = cadd(cmul(hmix.ck, kk), cmul(hmix.cw, w));
    k.g = cmul(hmix.cw, g);
    return k;
}

// Point data of one element at local (s,t): position, n~, a and, per local basis
// function, w*phi (component 0) and for the hypersingular part w*c with
// c = d_s phi F_t - d_t phi F_s (components 1..3).
template <int P, bool HARD>
__device__ __forceinline__ void point_data(const ElemRef& R, const double* Cu, const double* Cv, double s,
                                           double t, double w, double* g7, double* ph /*[NL][NV]*/) {
    constexpr int NV = HARD ? 4 : 1;
    GeoPt G;
    eval_geo(R.bez, R.pu, R.pv, s, t, G);
    double nt[3];
    cross3(G.fs, G.ft, nt);
    g7[0] = G.x[0]; g7[1] = G.x[1]; g7[2] = G.x[2];
    g7[3] = nt[0]; g7[4] = nt[1]; g7[5] = nt[2];
    g7[6] = sqrt(nt[0] * nt[0] + nt[1] * nt[1] + nt[2] * nt[2]);
    double bu[P + 1], bv[P + 1], dbu[P + 1], dbv[P + 1];
    eval_basis1<P>(Cu, s, bu, dbu);
    eval_basis1<P>(Cv, t, bv, dbv);
#pragma unroll
    for (int av = 0; av <= P; ++av)
#pragma unroll
        for (int au = 0; au <= P; ++au) {
            double* o = ph + (av * (P + 1) + au) * NV;
            o[0] = w * bv[av] * bu[au];
            if (HARD) {
                const double ds = bv[av] * dbu[au], dt = dbv[av] * bu[au];
#pragma unroll
                for (int c = 0; c < 3; ++c) o[1 + c] = w * (ds * G.ft[c] - dt * G.fs[c]);
            }
        }
}

// --------------------------------------------------------------------------
// Near field: regular element pairs, tensor Gauss rules of orders (nu, nv) on
// each element (nu * nv <= MAXQ points; the orders may differ between the two
// elements and between directions).  Kernel values are produced in chunks of
// CI test points in LDS; thread items (j, a) accumulate
// T[j][a] = sum_i w phi_a(x_i) k(x_i, y_j); finally B[a][b] = sum_j T[j][a] . w phi_b(y_j).
// --------------------------------------------------------------------------
template <int P, bool HARD, int MAXQ>
__global__ __launch_bounds__(NEAR_THREADS) void near_regular(NearArgs A) {
    constexpr int NL = (P + 1) * (P + 1);
    constexpr int NV = HARD ? 4 : 1;
    constexpr int NK = HARD ? 2 : 1;
    constexpr int CI = 8;
    constexpr int BUF = (CI * MAXQ * NK > MAXQ * NL) ? CI * MAXQ * NK : MAXQ * NL;
    constexpr int ITEMS = (MAXQ * NL + NEAR_THREADS - 1) / NEAR_THREADS;
    __shared__ double xg[MAXQ][7];
    __shared__ double yg[MAXQ][7];
    __shared__ double px[MAXQ][NL * NV];
    __shared__ double py[MAXQ][NL * NV];
    __shared__ double2 buf[BUF];

    const int64_t item = blockIdx.x;
    if (item >= A.nlist) return;
    const int k = A.list[item];
    const int e = A.pair_e[k], f = A.pair_f[k];
    const int kind = A.pair_kind[k];
    const int nxu = (kind >> 8) & 15, nxv = (kind >> 12) & 15, nyu = (kind >> 16) & 15, nyv = (kind >> 20) & 15;
    const int nx = nxu * nxv, ny = nyu * nyv;
    const int tid = threadIdx.x;

    if (tid < nx + ny) {
        const bool isx = tid < nx;
        const int i = isx ? tid : tid - nx;
        const int nu = isx ? nxu : nyu, nv = isx ? nxv : nyv;
        const double* gu = A.gl + nu * 2 * NGMAX;
        const double* gv = A.gl + nv * 2 * NGMAX;
        const ElemRef R = elem_ref(A.bez, A.pg, A.nel1, isx ? e : f);
        point_data<P, HARD>(R, A.C1 + R.ex * (P + 1) * (P + 1), A.C1 + R.ey * (P + 1) * (P + 1), gu[i % nu],
                            gv[i / nu], gu[NGMAX + i % nu] * gv[NGMAX + i / nu], isx ? xg[i] : yg[i],
                            isx ? px[i] : py[i]);
    }
    __syncthreads();

    double2 acc[ITEMS][NV];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it)
#pragma unroll
        for (int v = 0; v < NV; ++v) acc[it][v] = make_double2(0, 0);
    for (int i0 = 0; i0 < nx; i0 += CI) {
        const int ci = min(CI, nx - i0);
        for (int idx = tid; idx < ci * ny; idx += NEAR_THREADS) {
            const int i = i0 + idx / ny, j = idx % ny;
            const KVal kv = kernel_pair<HARD>(xg[i], xg[i] + 3, xg[i][6], yg[j], yg[j] + 3, yg[j][6], A.kappa, A.mix,
                                                 A.hmix);
            buf[idx * NK] = kv.s;
            if (HARD) buf[idx * NK + 1] = kv.g;
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const int w = tid + it * NEAR_THREADS;
            if (w < ny * NL) {
                const int j = w / NL, a = w % NL;
                for (int ii = 0; ii < ci; ++ii) {
                    const double* pxv = &px[i0 + ii][a * NV];
                    const double2 ks = buf[(ii * ny + j) * NK];
                    acc[it][0].x = fma(pxv[0], ks.x, acc[it][0].x);
                    acc[it][0].y = fma(pxv[0], ks.y, acc[it][0].y);
                    if (HARD) {
                        const double2 kg = buf[(ii * ny + j) * NK + 1];
#pragma unroll
                        for (int v = 1; v < NV; ++v) {
                            acc[it][v].x = fma(pxv[v], kg.x, acc[it][v].x);
                            acc[it][v].y = fma(pxv[v], kg.y, acc[it][v].y);
                        }
                    }
                }
            }
        }
        __syncthreads();
    }
    // one component v at a time: T[j][a] into LDS, then B[a][b] += sum_j T[j][a] py[j][b][v]
    // (keeps the buffer at MAXQ * NL entries, which the degree-3 hypersingular case needs)
    const int a = tid / NL, b = tid % NL;
    double2 sum = make_double2(0, 0);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const int w = tid + it * NEAR_THREADS;
            if (w < ny * NL) buf[w] = acc[it][v];
        }
        __syncthreads();
        if (tid < NL * NL)
            for (int j = 0; j < ny; ++j) {
                const double2 t = buf[j * NL + a];
                const double y = py[j][b * NV + v];
                sum.x = fma(t.x, y, sum.x);
                sum.y = fma(t.y, y, sum.y);
            }
        __syncthreads();
    }
    if (tid < NL * NL) A.stage[(int64_t(k) - A.slot0) * NL * NL + tid] = sum;
}

// --------------------------------------------------------------------------
// Near field: touching element pairs (Duffy-type rules on [0,1]^4), points in
// batches staged through LDS; output (a,b) accumulated by SPLIT threads each.
// --------------------------------------------------------------------------
template <int P, bool HARD>
__global__ __launch_bounds__(NEAR_THREADS) void near_singular(NearArgs A) {
    constexpr int NL = (P + 1) * (P + 1);
    constexpr int NV = HARD ? 4 : 1;
    constexpr int BATCH = HARD ? 64 : NEAR_THREADS;
    constexpr int SPLIT = NEAR_THREADS / (NL * NL) > 0 ? NEAR_THREADS / (NL * NL) : 1;
    __shared__ KVal kq[BATCH];
    __shared__ double px[BATCH][NL * NV];
    __shared__ double py[BATCH][NL * NV];
    __shared__ double2 red[NEAR_THREADS];

    const int64_t item = blockIdx.x;
    if (item >= A.nlist) return;
    const int k = A.list[item];
    const int e = A.pair_e[k], f = A.pair_f[k];
    const int kind = A.pair_kind[k];
    const int cls = kind & 15;
    const int te = (kind >> 16) & 7, tf = (kind >> 20) & 7;
    const int ri = cls == 4 ? 2 : cls == 2 ? 1 : 0;
    const double* rule = A.rule[ri];
    const int Q = A.rule_n[ri];
    const int tid = threadIdx.x;
    const ElemRef Re = elem_ref(A.bez, A.pg, A.nel1, e);
    const ElemRef Rf = elem_ref(A.bez, A.pg, A.nel1, f);
    const double* Ce_u = A.C1 + Re.ex * (P + 1) * (P + 1);
    const double* Ce_v = A.C1 + Re.ey * (P + 1) * (P + 1);
    const double* Cf_u = A.C1 + Rf.ex * (P + 1) * (P + 1);
    const double* Cf_v = A.C1 + Rf.ey * (P + 1) * (P + 1);

    const int out = tid % (NL * NL), part = tid / (NL * NL);
    const int oa = out / NL, ob = out % NL;
    double2 acc = make_double2(0, 0);
    for (int base = 0; base < Q; base += BATCH) {
        if (tid < BATCH) {
            const int qi = base + tid;
            if (qi < Q) {
                const double* r = rule + int64_t(qi) * 5;
                double s, t, u, v;
                d4_apply(te, r[0], r[1], s, t);
                d4_apply(tf, r[2], r[3], u, v);
                double gxv[7], gyv[7];
                point_data<P, HARD>(Re, Ce_u, Ce_v, s, t, 1.0, gxv, px[tid]);
                point_data<P, HARD>(Rf, Cf_u, Cf_v, u, v, 1.0, gyv, py[tid]);
                KVal kv = kernel_pair<HARD>(gxv, gxv + 3, gxv[6], gyv, gyv + 3, gyv[6], A.kappa, A.mix, A.hmix);
                kv.s = cscale(kv.s, r[4]);
                kv.g = cscale(kv.g, r[4]);
                kq[tid] = kv;
            } else {
                kq[tid].s = make_double2(0, 0);
                kq[tid].g = make_double2(0, 0);
#pragma unroll
                for (int a = 0; a < NL * NV; ++a) {
                    px[tid][a] = 0;
                    py[tid][a] = 0;
                }
            }
        }
        __syncthreads();
        if (part < SPLIT) {
            for (int q = part; q < BATCH; q += SPLIT) {
                const double w = px[q][oa * NV] * py[q][ob * NV];
                acc.x = fma(w, kq[q].s.x, acc.x);
                acc.y = fma(w, kq[q].s.y, acc.y);
                if (HARD) {
                    double c = 0;
#pragma unroll
                    for (int v = 1; v < NV; ++v) c = fma(px[q][oa * NV + v], py[q][ob * NV + v], c);
                    acc.x = fma(c, kq[q].g.x, acc.x);
                    acc.y = fma(c, kq[q].g.y, acc.y);
                }
            }
        }
        __syncthreads();
    }
    red[tid] = acc;
    __syncthreads();
    if (tid < NL * NL) {
        double2 sum = make_double2(0, 0);
        for (int g2 = 0; g2 < SPLIT; ++g2) sum = cadd(sum, red[g2 * NL * NL + tid]);
        if (cls == 4 && (A.cm.x != 0 || A.cm.y != 0)) {
            // + cm times the mass matrix on the identical pair: int phi_a phi_b a
            const int n = A.mass_order;
            const double* gx = A.gl + n * 2 * NGMAX;
            const double* gw = gx + NGMAX;
            double m = 0;
            for (int i = 0; i < n * n; ++i) {
                const double ss = gx[i % n], tt = gx[i / n];
                GeoPt G;
                eval_geo(Re.bez, Re.pu, Re.pv, ss, tt, G);
                double nt[3];
                cross3(G.fs, G.ft, nt);
                double bu[P + 1], bv[P + 1];
                eval_basis1<P>(Ce_u, ss, bu, nullptr);
                eval_basis1<P>(Ce_v, tt, bv, nullptr);
                const double pa = bv[oa / (P + 1)] * bu[oa % (P + 1)];
                const double pb = bv[ob / (P + 1)] * bu[ob % (P + 1)];
                m += gw[i % n] * gw[i / n] * sqrt(nt[0] * nt[0] + nt[1] * nt[1] + nt[2] * nt[2]) * pa * pb;
            }
            sum.x += A.cm.x * m;
            sum.y += A.cm.y * m;
        }
        A.stage[(int64_t(k) - A.slot0) * NL * NL + tid] = sum;
    }
}

// --------------------------------------------------------------------------
// Near field: deterministic gather of the staged element blocks into the CSR
// values of the solution space.  One workgroup per row; each nonzero sums its
// contributions in a fixed order (representatives, elements, source elements).
// --------------------------------------------------------------------------
struct CsrArgs {
    const int64_t* row_ptr;
    const int* col;
    double2* val;
    const int64_t* near_ptr;
    const int* near_src;
    const double2* stage;
    int64_t slot0;
    int64_t e_lo, e_hi;          // target elements whose pairs are staged
    const int* s0_ptr;           // null for S^2 (soft)
    const int* s0_reps;
    int64_t row0;
    int nel1, k;
};

template <int P>
__global__ void near_gather_csr(CsrArgs A) {
    constexpr int NL = (P + 1) * (P + 1);
    const int64_t row = A.row0 + blockIdx.x;
    const int64_t beg = A.row_ptr[row], end = A.row_ptr[row + 1];
    const int64_t kk = int64_t(A.k) * A.k;
    const int r0 = A.s0_ptr ? A.s0_ptr[row] : int(row);
    const int r1 = A.s0_ptr ? A.s0_ptr[row + 1] : int(row) + 1;
    for (int64_t idx = beg + threadIdx.x; idx < end; idx += blockDim.x) {
        const int colv = A.col[idx];
        const int c0 = A.s0_ptr ? A.s0_ptr[colv] : colv;
        const int c1 = A.s0_ptr ? A.s0_ptr[colv + 1] : colv + 1;
        double2 acc = make_double2(0, 0);
        for (int ri = r0; ri < r1; ++ri) {
            const int64_t i = A.s0_ptr ? A.s0_reps[ri] : ri;
            const int pj = int(i / kk), rem = int(i % kk), iv = rem / A.k, iu = rem % A.k;
            for (int ey = max(0, iv - P); ey <= min(iv, A.nel1 - 1); ++ey)
                for (int ex = max(0, iu - P); ex <= min(iu, A.nel1 - 1); ++ex) {
                    const int64_t e = (int64_t(pj) * A.nel1 + ey) * A.nel1 + ex;
                    if (e < A.e_lo || e >= A.e_hi) continue;
                    const int a = (iv - ey) * (P + 1) + (iu - ex);
                    const int64_t nb = A.near_ptr[e], ne = A.near_ptr[e + 1];
                    for (int ci = c0; ci < c1; ++ci) {
                        const int64_t j = A.s0_ptr ? A.s0_reps[ci] : ci;
                        const int qj = int(j / kk), rj = int(j % kk), jv = rj / A.k, ju = rj % A.k;
                        for (int fy = max(0, jv - P); fy <= min(jv, A.nel1 - 1); ++fy)
                            for (int fx = max(0, ju - P); fx <= min(ju, A.nel1 - 1); ++fx) {
                                const int f = int((int64_t(qj) * A.nel1 + fy) * A.nel1 + fx);
                                int64_t lo = nb, hi = ne;
                                while (lo < hi) {
                                    int64_t mid = (lo + hi) >> 1;
                                    if (A.near_src[mid] < f) lo = mid + 1;
                                    else hi = mid;
                                }
                                if (lo < ne && A.near_src[lo] == f) {
                                    const int b = (jv - fy) * (P + 1) + (ju - fx);
                                    acc = cadd(acc, A.stage[(lo - A.slot0) * NL * NL + a * NL + b]);
                                }
                            }
                    }
                }
        }
        A.val[idx] = cadd(A.val[idx], acc);
    }
}

// ==========================================================================
// host launchers
// ==========================================================================
std::vector<double> gauss_table() {
    // Gauss-Legendre nodes / weights on [0,1] for orders 1..NGMAX by Newton's
    // iteration on the Legendre recurrence
    std::vector<double> t((NGMAX + 1) * 2 * NGMAX, 0.0);
    for (int n = 1; n <= NGMAX; ++n) {
        for (int i = 0; i < n; ++i) {
            double x = std::cos(M_PI * (i + 0.75) / (n + 0.5));
            double dp = 1;
            for (int it = 0; it < 100; ++it) {
                double p0 = 1, p1 = x;
                for (int k = 2; k <= n; ++k) {
                    double p2 = ((2 * k - 1) * x * p1 - (k - 1) * p0) / k;
                    p0 = p1;
                    p1 = p2;
                }
                if (n == 1) { p1 = x; p0 = 1; }
                dp = n * (x * p1 - p0) / (x * x - 1);
                double dx = p1 / dp;
                x -= dx;
                if (std::fabs(dx) < 1e-16) break;
            }
            double p0 = 1, p1 = x;
            for (int k = 2; k <= n; ++k) {
                double p2 = ((2 * k - 1) * x * p1 - (k - 1) * p0) / k;
                p0 = p1;
                p1 = p2;
            }
            dp = n * (x * p1 - p0) / (x * x - 1);
            t[n * 2 * NGMAX + i] = 0.5 * (1 - x);
            t[n * 2 * NGMAX + NGMAX + i] = 1.0 / ((1 - x * x) * dp * dp);
        }
    }
    return t;
}

void gauss01_host(int n, std::vector<double>& x, std::vector<double>& w) {
    static std::vector<double> tab = gauss_table();
    n = std::max(1, std::min(n, NGMAX));
    x.assign(tab.begin() + n * 2 * NGMAX, tab.begin() + n * 2 * NGMAX + n);
    w.assign(tab.begin() + n * 2 * NGMAX + NGMAX, tab.begin() + n * 2 * NGMAX + NGMAX + n);
}

namespace {

// Duffy-type rules on [0,1]^4 as (s1, s2, r1, r2, w) for the three touching
// configurations (identical element; shared edge s2 = r2 = 0 with s1 = r1;
// shared vertex at the origin).  Each coordinate pair (s, r) of the identical
// and edge cases is written as offset u = |r - s| and position w in [0,1]
// (Jacobian 1 - u); the singular corner of the remaining cube is removed by
// splitting it into simplices / pyramids along its largest coordinate rho.
std::vector<double> duffy_rule(int cls, int n) {
    std::vector<double> gx, gw;
    gauss01_host(n, gx, gw);
    std::vector<double> out;
    auto split = [](double u, double w, int sig, double& s, double& r) {
        double base = w * (1 - u);
        if (sig > 0) { s = base; r = base + u; }
        else { s = base + u; r = base; }
    };
    for (int a = 0; a < n; ++a)
        for (int b = 0; b < n; ++b)
            for (int c = 0; c < n; ++c)
                for (int d = 0; d < n; ++d) {
                    const double rho = gx[a], t1 = gx[b], t2 = gx[c], t3 = gx[d];
                    const double W = gw[a] * gw[b] * gw[c] * gw[d];
                    if (cls == 2) {  // identical: 2 x 2 signs x 2 triangles
                        for (int sg = 0; sg < 4; ++sg)
                            for (int tri = 0; tri < 2; ++tri) {
                                double u1 = tri ? rho * t1 : rho, u2 = tri ? rho : rho * t1;
                                double s1, r1, s2, r2;
                                split(u1, t2, (sg & 1) ? -1 : 1, s1, r1);
                                split(u2, t3, (sg & 2) ? -1 : 1, s2, r2);
                                out.insert(out.end(), {s1, s2, r1, r2, W * (1 - u1) * (1 - u2) * rho});
                            }
                    } else if (cls == 1) {  // edge: 2 signs x 3 pyramids
                        for (int sg = 0; sg < 2; ++sg)
                            for (int pyr = 0; pyr < 3; ++pyr) {
                                double u1, s2, r2;
                                if (pyr == 0) { u1 = rho; s2 = rho * t1; r2 = rho * t2; }
                                else if (pyr == 1) { u1 = rho * t1; s2 = rho; r2 = rho * t2; }
                                else { u1 = rho * t1; s2 = rho * t2; r2 = rho; }
                                double s1, r1;
                                split(u1, t3, sg ? -1 : 1, s1, r1);
                                out.insert(out.end(), {s1, s2, r1, r2, W * (1 - u1) * rho * rho});
                            }
                    } else {  // vertex: 4 pyramids
                        for (int pyr = 0; pyr < 4; ++pyr) {
                            double c4[4];
                            double rest[3] = {rho * t1, rho * t2, rho * t3};
                            for (int i = 0, j = 0; i < 4; ++i) c4[i] = (i == pyr) ? rho : rest[j++];
                            out.insert(out.end(), {c4[0], c4[1], c4[2], c4[3], W * rho * rho * rho});
                        }
                    }
                }
    return out;
}

}  // namespace

// orders of the GPU rules (see near_classify for the regular ones)
constexpr int NSING_IDENT = 7, NSING_EDGE = 8, NSING_VERTEX = 9, MASS_ORDER = 6;

template <int P, bool HARD>
static igb_status near_launch(igb_op op, hipStream_t s) {
    igb_geom g = op->geom;
    constexpr int NL = (P + 1) * (P + 1);
    const int64_t E = g->nelem;
    const int64_t npairs = op->near_ptr[E];
    size_t* acct = &op->dev_bytes;
    igb_status st;
    // pair arrays
    std::vector<int> pe(npairs);
    for (int64_t e = 0; e < E; ++e)
        for (int64_t k = op->near_ptr[e]; k < op->near_ptr[e + 1]; ++k) pe[k] = int(e);
    DevBuf d_pe, d_pf, d_kind, d_gl, d_rules[3], d_list, d_stage;
    if ((st = upload(d_pe, pe.data(), pe.size(), nullptr))) return st;
    if ((st = upload(d_pf, op->near_src.data(), op->near_src.size(), nullptr))) return st;
    if ((st = upload(d_kind, op->near_kind.data(), op->near_kind.size(), nullptr))) return st;
    std::vector<double> gl = gauss_table();
    if ((st = upload(d_gl, gl.data(), gl.size(), nullptr))) return st;
    const int raise = op->prm.quad_extra + kd_boost(op->kd_elem) + aspect_boost(op->aspect_max);
    const int ord[3] = {std::min(NGMAX, NSING_VERTEX + raise), std::min(NGMAX, NSING_EDGE + raise),
                        std::min(NGMAX, NSING_IDENT + raise)};
    NearArgs A{};
    for (int c = 0; c < 3; ++c) {
        std::vector<double> r = duffy_rule(c, ord[c]);
        if ((st = upload(d_rules[c], r.data(), r.size(), nullptr))) return st;
        A.rule[c] = d_rules[c].as<double>();
        A.rule_n[c] = int(r.size() / 5);
    }
    if ((st = upload(op->d_near_ptr, op->near_ptr.data(), op->near_ptr.size(), acct))) return st;
    if ((st = upload(op->d_near_src, op->near_src.data(), op->near_src.size(), acct))) return st;
    if ((st = upload(op->d_rowptr, op->row_ptr.data(), op->row_ptr.size(), acct))) return st;
    if ((st = upload(op->d_col, op->col.data(), op->col.size(), acct))) return st;
    if ((st = upload(op->d_dcol, op->near_dcol.data(), op->near_dcol.size(), acct))) return st;
    if ((st = upload(op->d_row_coff, op->row_coff.data(), op->row_coff.size(), acct))) return st;
    if ((st = upload(op->d_near_wgs, op->near_wgs.data(), op->near_wgs.size(), acct))) return st;
    if ((st = upload(op->d_near_grp_rows, op->near_grp_rows.data(), op->near_grp_rows.size(), acct))) return st;
    if ((st = alloc(op->d_val, op->nnz * sizeof(double2), acct))) return st;
    IGB_HIP(hipMemsetAsync(op->d_val.ptr, 0, op->nnz * sizeof(double2), s));

    A.bez = g->d_bez.as<double>();
    A.pg = g->d_pg.as<int>();
    A.C1 = g->d_C1.as<double>();
    A.gl = d_gl.as<double>();
    A.pair_e = d_pe.as<int>();
    A.pair_f = d_pf.as<int>();
    A.pair_kind = d_kind.as<int>();
    A.nel1 = g->nel1;
    A.kappa = op->kappa;
    A.eta = op->eta;
    A.mix = op->mix;
    A.hmix = op->hmix;
    A.cm = op->cm;
    A.mass_order = MASS_ORDER;

    // chunks of target elements with a bounded staging buffer
    const int64_t max_slots = std::max<int64_t>(int64_t(1) << 22, 1);  // 4M pairs
    if ((st = alloc(d_stage, size_t(std::min(npairs, max_slots)) * NL * NL * sizeof(double2), nullptr)))
        return st;
    if ((st = alloc(d_list, size_t(std::min(npairs, max_slots)) * sizeof(int), nullptr))) return st;
    A.stage = d_stage.as<double2>();
    const bool hard = op->bc == IGB_HARD;
    int64_t e0 = 0;
    std::vector<int> reg, reg_big, sing;
    auto points = [](int kind) {
        return std::max(((kind >> 8) & 15) * ((kind >> 12) & 15), ((kind >> 16) & 15) * ((kind >> 20) & 15));
    };
    while (e0 < E) {
        int64_t e1 = e0;
        while (e1 < E && op->near_ptr[e1 + 1] - op->near_ptr[e0] <= max_slots) ++e1;
        if (e1 == e0) {
            set_error("assemble_nearfield: one element has more near pairs than the staging buffer");
            return IGB_ERR_UNSUPPORTED;
        }
        const int64_t k0 = op->near_ptr[e0], k1 = op->near_ptr[e1];
        reg.clear();
        reg_big.clear();
        sing.clear();
        for (int64_t k = k0; k < k1; ++k) {
            const int kind = op->near_kind[k];
            ((kind & 15) != 0 ? sing : points(kind) <= 49 ? reg : reg_big).push_back(int(k));
        }
        A.slot0 = k0;
        // regular pairs with at most 49 points per element, then the larger regular
        // rules, then the touching pairs
        std::vector<int> lst(reg);
        lst.insert(lst.end(), reg_big.begin(), reg_big.end());
        lst.insert(lst.end(), sing.begin(), sing.end());
        if (!lst.empty())
            IGB_HIP(hipMemcpyAsync(d_list.ptr, lst.data(), lst.size() * sizeof(int), hipMemcpyHostToDevice, s));
        if (!reg.empty()) {
            A.list = d_list.as<int>();
            A.nlist = int64_t(reg.size());
            hipLaunchKernelGGL((near_regular<P, HARD, 49>), dim3(unsigned(reg.size())), dim3(NEAR_THREADS), 0, s, A);
            IGB_HIP(hipGetLastError());
        }
        if (!reg_big.empty()) {
            A.list = d_list.as<int>() + reg.size();
            A.nlist = int64_t(reg_big.size());
            hipLaunchKernelGGL((near_regular<P, HARD, REG_POINTS_MAX>), dim3(unsigned(reg_big.size())),
                               dim3(NEAR_THREADS), 0, s, A);
            IGB_HIP(hipGetLastError());
        }
        if (!sing.empty()) {
            A.list = d_list.as<int>() + reg.size() + reg_big.size();
            A.nlist = int64_t(sing.size());
            hipLaunchKernelGGL((near_singular<P, HARD>), dim3(unsigned(sing.size())), dim3(NEAR_THREADS), 0, s, A);
            IGB_HIP(hipGetLastError());
        }
        // rows touched by the chunk's target elements
        int64_t rlo = op->N, rhi = -1;
        for (int64_t e = e0; e < e1; ++e) {
            const int nel1 = g->nel1, k = g->k;
            int j = int(e / (int64_t(nel1) * nel1));
            int rem = int(e % (int64_t(nel1) * nel1));
            int ey = rem / nel1, ex = rem % nel1;
            for (int av = 0; av <= P; ++av)
                for (int au = 0; au <= P; ++au) {
                    int64_t i2 = (int64_t(j) * k + ey + av) * k + ex + au;
                    int64_t r = hard ? g->s2_to_s0[i2] : i2;
                    rlo = std::min(rlo, r);
                    rhi = std::max(rhi, r);
                }
        }
        CsrArgs C{};
        C.row_ptr = op->d_rowptr.as<int64_t>();
        C.col = op->d_col.as<int>();
        C.val = op->d_val.as<double2>();
        C.near_ptr = op->d_near_ptr.as<int64_t>();
        C.near_src = op->d_near_src.as<int>();
        C.stage = d_stage.as<double2>();
        C.slot0 = k0;
        C.e_lo = e0;
        C.e_hi = e1;
        C.s0_ptr = hard ? op->d_s0_ptr.as<int>() : nullptr;
        C.s0_reps = hard ? op->d_s0_reps.as<int>() : nullptr;
        C.row0 = rlo;
        C.nel1 = g->nel1;
        C.k = g->k;
        if (rhi >= rlo) {
            hipLaunchKernelGGL(near_gather_csr<P>, dim3(unsigned(rhi - rlo + 1)), dim3(256), 0, s, C);
            IGB_HIP(hipGetLastError());
        }
        IGB_HIP(hipStreamSynchronize(s));
        e0 = e1;
    }
    return IGB_OK;
}

igb_status near_field_device(igb_op op, hipStream_t s) {
    const bool hard = op->bc == IGB_HARD;
    return with_degree(op->geom->p, "assemble_nearfield", [&](auto deg) {
        constexpr int P = decltype(deg)::value;
        if constexpr (P == 0)
            return near_launch<0, false>(op, s);  // S^0 needs p >= 1: checked at the entry point
        else
            return hard ? near_launch<P, true>(op, s) : near_launch<P, false>(op, s);
    });
}

}  // namespace igb

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
constexpr int MASS_ORDER = 6;   // Gauss order per direction of the mass matrix on identical pairs

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
    // touching-pair rules per class (0 vertex, 1 edge, 2 identical): blocks of 10
    // doubles (duffy_blocks) and the Gauss order n of the tensor grid in each block
    const double* rule[3];
    int rule_n[3];     // blocks
    int rule_ord[3];   // n
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
    const double d0 = X[0] - Y[0], d1 = X[1] - Y[1], d2 = X[2] - Y[2];
    const double r2 = d0 * d0 + d1 * d1 + d2 * d2;
    const double ir = rsqrt_fast(r2);
    const double kr = kappa * (r2 * ir);
    double sn, cs;
    sincos_fast(kr, sn, cs);
    const double c4 = 0.07957747154594767 * ir;   // 1/(4 pi r)
    if (!HARD) {
        // ck a_y H (x-y).n~_x + cv a_x a_y G as in kernel_soft
        const double dn = d0 * NX[0] + d1 * NX[1] + d2 * NX[2];
        const double h = mix.ck * ay * dn * ir * ir * c4, v = ax * ay * c4;
        k.s = make_double2(h * (-cs - sn * kr) + v * (mix.cv.x * cs - mix.cv.y * sn),
                           h * (cs * kr - sn) + v * (mix.cv.x * sn + mix.cv.y * cs));
        k.g = make_double2(0, 0);
        return k;
    }
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
// Near field: touching element pairs (Duffy-type rules on [0,1]^4, duffy_blocks).
//
// In every region of the rules the point (s1, s2; r1, r2) of a block (the outer
// variables fixed) runs over an n x n tensor grid on which (s1, r1) depend on
// the first grid index alone and (s2, r2) on the second alone, all affinely in
// the Gauss node.  So with Bernstein polynomials b on the elements, the block's
// contribution factorises:
//   sum_beta [b_j(s2) b_l(r2)]_beta  sum_alpha [b_i(s1) b_k(r1)]_alpha K(alpha, beta).
// A lane takes a line (block, beta): it contracts both control nets along the
// line's fixed coordinate once, walks alpha (two rational curve points and one
// kernel value per point pair) and sums the (p+1)^2 products of the inner
// factor; 64 lines then meet their outer factors on the fp64 matrix cores.  The
// B-spline extraction is applied once per pair, to the finished matrix.  The
// element symmetries of the rule are put into the nets and extraction rows as
// they are read, so the grid is the same for every pair.
// (Sound-hard: the curl product c_a . c_b, c = d1 phi F_2 - d2 phi F_1, splits into
// four factorised terms with the kernel times F_i.F_j; the first shares the
// outer factor of the phi phi term.)
// Bound by fp64 VALU issue: about 250 instructions per point pair (sound-hard
// about 450), where the point-wise form needed two surface points and (p+1)^4
// products per point pair.  Level 5, p = 2, 55 thousand pairs (1.37 10^9 point
// pairs): 79 -> 17 ms sound-soft, 287 -> 37.5 ms sound-hard (the sound-hard form
// keeps 72 accumulators and runs one wave per SIMD).
// --------------------------------------------------------------------------
// wavefront-wide ordering of LDS traffic inside one wave
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
typedef double f64x4 __attribute__((ext_vector_type(4)));

// Bernstein polynomials of compile-time degree
template <int P>
__device__ __forceinline__ void bern(double s, double* b) {
    double db[4];
    bernstein(P, s, b, db);
}

// entry (k, i) of the degree elevation from p to q >= p: b^q_k = sum_i E(k, i) b^p_i
__device__ __forceinline__ double elevation(int p, int q, int k, int i) {
    constexpr double C[4][4] = {{1, 0, 0, 0}, {1, 1, 0, 0}, {1, 2, 1, 0}, {1, 3, 3, 1}};
    const int r = k - i;
    return r < 0 || r > q - p ? 0.0 : C[p][i] * C[q - p][r] / C[q][k];
}

// P: spline degree, G >= the geometry degree of every element (lower degrees are
// elevated as the net is read)
template <int P, bool HARD, int G>
__global__ __launch_bounds__(NEAR_THREADS, !HARD && P <= 2 ? 2 : 1) void near_singular(NearArgs A) {
    constexpr int P1 = P + 1, NL = P1 * P1, G1 = G + 1, NW = NEAR_THREADS / 64;
    constexpr int NT = HARD ? 4 : 1;   // factorised terms with their own outer factor
    __shared__ double net[2][G1][G1][4];      // [x, y][dim 1][dim 2][homogeneous]
    __shared__ double ext[2][2][P1][P1];      // [x, y][dim][B-spline][Bernstein]
    __shared__ double2 Tb[NW][64][NL];        // a chunk's inner sums, one term at a time
    __shared__ double Qb[NW][64][NL];         // and its outer factors
    __shared__ double2 Mb[NL][NL], Rb[NL][NL];
    __shared__ double mw[MASS_ORDER * MASS_ORDER], mb[MASS_ORDER * MASS_ORDER * 2 * P1];   // mass matrix points
    double2* red = &Tb[0][0][0];              // [NW][NL][NL] after the loop
    static_assert(sizeof(double2) * NW * NL * NL <= sizeof(Tb), "the waves' sums fit");

    const int64_t item = blockIdx.x;
    if (item >= A.nlist) return;
    const int kp = A.list[item];
    const int kind = A.pair_kind[kp];
    const int cls = kind & 15;
    const int ri = cls == 4 ? 2 : cls == 2 ? 1 : 0;
    const double* rule = A.rule[ri];
    const int n = A.rule_ord[ri], nlines = A.rule_n[ri] * n;
    const double* gx = A.gl + n * 2 * NGMAX;
    const double* gw = gx + NGMAX;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, g = lane >> 4;
    const int code[2] = {(kind >> 16) & 7, (kind >> 20) & 7};
    const ElemRef R[2] = {elem_ref(A.bez, A.pg, A.nel1, A.pair_e[kp]), elem_ref(A.bez, A.pg, A.nel1, A.pair_f[kp])};

    // canonical nets and extraction rows (dim 1 = u unless swapped; flips reverse)
    for (int t = tid; t < 2 * G1 * G1 * 4; t += NEAR_THREADS) {
        const int x = t / (G1 * G1 * 4), r = t % (G1 * G1 * 4), i = r / (G1 * 4), j = (r / 4) % G1, c = r % 4;
        const int cd = code[x];
        int iu = (cd & 4) ? j : i, iv = (cd & 4) ? i : j;
        if (cd & 1) iu = G - iu;
        if (cd & 2) iv = G - iv;
        const int pu = R[x].pu, pv = R[x].pv;
        double v = 0;
        for (int b = 0; b <= pv; ++b)
            for (int a = 0; a <= pu; ++a)
                v = fma(elevation(pu, G, iu, a) * elevation(pv, G, iv, b), R[x].bez[(b * (PGMAX + 1) + a) * 4 + c], v);
        net[x][i][j][c] = v;
    }
    for (int t = tid; t < 4 * P1 * P1; t += NEAR_THREADS) {
        const int x = t / (2 * P1 * P1), dim = (t / (P1 * P1)) & 1, a = (t / P1) % P1, k = t % P1;
        const int cd = code[x];
        const bool along_u = (dim == 0) == !(cd & 4);
        const bool flip = along_u ? (cd & 1) : (cd & 2);
        const double* C = A.C1 + (along_u ? R[x].ex : R[x].ey) * P1 * P1;
        ext[x][dim][a][k] = C[a * P1 + (flip ? P - k : k)];
    }
    // orientation of the canonical coordinates: n~ and the curls change sign with
    // every swap or flip
    double sg[2];
#pragma unroll
    for (int x = 0; x < 2; ++x) sg[x] = (__popc(code[x]) & 1) ? -1.0 : 1.0;
    const double sxy = sg[0] * sg[1];
    __syncthreads();

    f64x4 accr = {0, 0, 0, 0}, acci = {0, 0, 0, 0};
    for (int l0 = wave * 64; l0 < nlines; l0 += NW * 64) {
        // this lane's line; lanes past the last repeat it with weight 0
        const int ln = min(l0 + lane, nlines - 1), o = ln / n, be = ln % n;
        const double* B = rule + int64_t(o) * 10;
        const double a1 = B[0], b1 = B[1], c1 = B[2], d1 = B[3];
        const double s2 = fma(B[5], gx[be], B[4]), r2 = fma(B[7], gx[be], B[6]);
        const double wl = l0 + lane < nlines ? B[8] * gw[be] : 0.0;
        double q[2][G1][4], dq[2][G1][4];   // nets contracted along dim 2: values, d/d dim 2
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            double bb[4], db[4];
            bernstein(G, x ? r2 : s2, bb, db);
#pragma unroll
            for (int i = 0; i < G1; ++i)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    double v = 0, d = 0;
#pragma unroll
                    for (int j = 0; j < G1; ++j) {
                        const double h = net[x][i][j][c];
                        v = fma(bb[j], h, v);
                        d = fma(db[j], h, d);
                    }
                    q[x][i][c] = v;
                    dq[x][i][c] = d;
                }
        }
        double2 T[NT][P1][P1];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < P1; ++i)
#pragma unroll
                for (int k = 0; k < P1; ++k) T[t][i][k] = make_double2(0, 0);
        for (int al = 0; al < n; ++al) {
            const double ga = gx[al], wa = gw[al];
            const double st[2] = {fma(b1, ga, a1), fma(d1, ga, c1)};
            double X[2][3], F1[2][3], F2[2][3], N[2][3], ar[2];
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                double bb[4], db[4];
                bernstein(G, st[x], bb, db);
                double p0[4], p1[4], p2[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    p0[c] = bb[0] * q[x][0][c];
                    p1[c] = db[0] * q[x][0][c];
                    p2[c] = bb[0] * dq[x][0][c];
#pragma unroll
                    for (int i = 1; i < G1; ++i) {
                        p0[c] = fma(bb[i], q[x][i][c], p0[c]);
                        p1[c] = fma(db[i], q[x][i][c], p1[c]);
                        p2[c] = fma(bb[i], dq[x][i][c], p2[c]);
                    }
                }
                const double iw = rcp_fast(p0[3]);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    X[x][c] = p0[c] * iw;
                    F1[x][c] = (p1[c] - X[x][c] * p1[3]) * iw;
                    F2[x][c] = (p2[c] - X[x][c] * p2[3]) * iw;
                }
                cross3(F1[x], F2[x], N[x]);
#pragma unroll
                for (int c = 0; c < 3; ++c) N[x][c] *= sg[x];
                const double n2 = N[x][0] * N[x][0] + N[x][1] * N[x][1] + N[x][2] * N[x][2];
                ar[x] = n2 * rsqrt_fast(n2);
            }
            const KVal kv = kernel_pair<HARD>(X[0], N[0], ar[0], X[1], N[1], ar[1], A.kappa, A.mix, A.hmix);
            const double2 S = cscale(kv.s, wa);
            double bx[4], dbx[4], by[4], dby[4];
            bernstein(P, st[0], bx, dbx);
            bernstein(P, st[1], by, dby);
#pragma unroll
            for (int i = 0; i < P1; ++i) {
                const double2 u = cscale(S, bx[i]);
#pragma unroll
                for (int k = 0; k < P1; ++k) {
                    T[0][i][k].x = fma(u.x, by[k], T[0][i][k].x);
                    T[0][i][k].y = fma(u.y, by[k], T[0][i][k].y);
                }
            }
            if constexpr (HARD) {
                const double2 Gw = cscale(kv.g, wa * sxy);
                const double e22 = F2[0][0] * F2[1][0] + F2[0][1] * F2[1][1] + F2[0][2] * F2[1][2];
                const double e21 = F2[0][0] * F1[1][0] + F2[0][1] * F1[1][1] + F2[0][2] * F1[1][2];
                const double e12 = F1[0][0] * F2[1][0] + F1[0][1] * F2[1][1] + F1[0][2] * F2[1][2];
                const double e11 = F1[0][0] * F1[1][0] + F1[0][1] * F1[1][1] + F1[0][2] * F1[1][2];
                const double2 g22 = cscale(Gw, e22), g21 = cscale(Gw, -e21), g12 = cscale(Gw, -e12), g11 = cscale(Gw, e11);
#pragma unroll
                for (int i = 0; i < P1; ++i) {
                    const double2 u0 = cscale(g22, dbx[i]), u1 = cscale(g21, dbx[i]), u2 = cscale(g12, bx[i]),
                                  u3 = cscale(g11, bx[i]);
#pragma unroll
                    for (int k = 0; k < P1; ++k) {
                        T[0][i][k].x = fma(u0.x, dby[k], T[0][i][k].x);
                        T[0][i][k].y = fma(u0.y, dby[k], T[0][i][k].y);
                        T[1][i][k].x = fma(u1.x, by[k], T[1][i][k].x);
                        T[1][i][k].y = fma(u1.y, by[k], T[1][i][k].y);
                        T[2][i][k].x = fma(u2.x, dby[k], T[2][i][k].x);
                        T[2][i][k].y = fma(u2.y, dby[k], T[2][i][k].y);
                        T[3][i][k].x = fma(u3.x, by[k], T[3][i][k].x);
                        T[3][i][k].y = fma(u3.y, by[k], T[3][i][k].y);
                    }
                }
            }
        }
        // outer factors (weighted): b_j b_l, and sound-hard b_j d_l, d_j b_l, d_j d_l
        double bx[4], dbx[4], by[4], dby[4];
        bernstein(P, s2, bx, dbx);
        bernstein(P, r2, by, dby);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            wave_lds_sync();   // the previous term's operands are read
#pragma unroll
            for (int i = 0; i < P1; ++i)
#pragma unroll
                for (int k = 0; k < P1; ++k) {
                    Tb[wave][lane][i * P1 + k] = T[t][i][k];
                    Qb[wave][lane][i * P1 + k] = wl * (t < 2 ? bx[i] : dbx[i]) * (t == 0 || t == 2 ? by[k] : dby[k]);
                }
            wave_lds_sync();
            // rows: outer index (j, l); columns: inner index (i, k); rows and columns
            // past NL repeat the last and are not read
            const int lc = min(li, NL - 1);
#pragma unroll
            for (int st = 0; st < 16; ++st) {
                const double Aq = Qb[wave][4 * st + g][lc];
                const double2 Bt = Tb[wave][4 * st + g][lc];
                accr = __builtin_amdgcn_mfma_f64_16x16x4f64(Aq, Bt.x, accr, 0, 0, 0);
                acci = __builtin_amdgcn_mfma_f64_16x16x4f64(Aq, Bt.y, acci, 0, 0, 0);
            }
        }
    }
    // the waves' sums meet in wave order
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int jl = g + 4 * r;
        if (jl < NL && li < NL) red[(wave * NL + jl) * NL + li] = make_double2(accr[r], acci[r]);
    }
    __syncthreads();
    if (tid < NL * NL) {
        double2 s = red[tid];
#pragma unroll
        for (int w = 1; w < NW; ++w) s = cadd(s, red[w * NL * NL + tid]);
        Mb[tid / NL][tid % NL] = s;
    }
    __syncthreads();
    // extraction along dim 1: R[jl][a1 b1], then along dim 2
    if (tid < NL * NL) {
        const int jl = tid / NL, a1i = (tid % NL) / P1, b1i = tid % P1;
        double2 s = make_double2(0, 0);
        for (int i = 0; i < P1; ++i)
            for (int k = 0; k < P1; ++k) {
                const double f = ext[0][0][a1i][i] * ext[1][0][b1i][k];
                const double2 m = Mb[jl][i * P1 + k];
                s.x = fma(f, m.x, s.x);
                s.y = fma(f, m.y, s.y);
            }
        Rb[jl][tid % NL] = s;
    }
    // mass matrix of identical pairs (element coordinates): points' weight times
    // measure and basis values
    const bool mass = cls == 4 && (A.cm.x != 0 || A.cm.y != 0);
    constexpr int nm = MASS_ORDER;
    if (mass && tid < nm * nm) {
        const double* mx = A.gl + nm * 2 * NGMAX;
        const double ss = mx[tid % nm], tt = mx[tid / nm];
        GeoPt gp;
        eval_geo(R[0].bez, R[0].pu, R[0].pv, ss, tt, gp);
        double nt[3];
        cross3(gp.fs, gp.ft, nt);
        mw[tid] = mx[NGMAX + tid % nm] * mx[NGMAX + tid / nm] * sqrt(nt[0] * nt[0] + nt[1] * nt[1] + nt[2] * nt[2]);
        eval_basis1<P>(A.C1 + R[0].ex * P1 * P1, ss, mb + tid * 2 * P1, nullptr);
        eval_basis1<P>(A.C1 + R[0].ey * P1 * P1, tt, mb + tid * 2 * P1 + P1, nullptr);
    }
    __syncthreads();
    if (tid < NL * NL) {
        // output (a, b): element-local indices (v major) to canonical ones
        const int oa = tid / NL, ob = tid % NL;
        const int a1i = (code[0] & 4) ? oa / P1 : oa % P1, a2i = (code[0] & 4) ? oa % P1 : oa / P1;
        const int b1i = (code[1] & 4) ? ob / P1 : ob % P1, b2i = (code[1] & 4) ? ob % P1 : ob / P1;
        double2 s = make_double2(0, 0);
        for (int j = 0; j < P1; ++j)
            for (int l = 0; l < P1; ++l) {
                const double f = ext[0][1][a2i][j] * ext[1][1][b2i][l];
                const double2 m = Rb[j * P1 + l][a1i * P1 + b1i];
                s.x = fma(f, m.x, s.x);
                s.y = fma(f, m.y, s.y);
            }
        if (mass) {
            double m = 0;
            for (int i = 0; i < nm * nm; ++i) {
                const double* u = mb + i * 2 * P1;
                m = fma(mw[i] * (u[P1 + oa / P1] * u[oa % P1]), u[P1 + ob / P1] * u[ob % P1], m);
            }
            s.x += A.cm.x * m;
            s.y += A.cm.y * m;
        }
        A.stage[(int64_t(kp) - A.slot0) * NL * NL + tid] = s;
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

// Duffy-type rules on [0,1]^4 for the three touching configurations (cls 2:
// identical element; 1: shared edge s2 = r2 = 0 with s1 = r1; 0: shared vertex at
// the origin).  Each coordinate pair (s, r) of the identical and edge cases is
// written as offset u = |r - s| and position w in [0,1] (Jacobian 1 - u); the
// singular corner of the remaining cube is removed by splitting it into
// simplices / pyramids along its largest coordinate rho.  As blocks of 10
// doubles over the n x n Gauss grid (x_alpha, x_beta):
//   s1 = B0 + B1 x_alpha, r1 = B2 + B3 x_alpha, s2 = B4 + B5 x_beta,
//   r2 = B6 + B7 x_beta, weight B8 w_alpha w_beta  (B9 unused)
std::vector<double> duffy_blocks(int cls, int n) {
    std::vector<double> gx, gw;
    gauss01_host(n, gx, gw);
    std::vector<double> out;
    struct Pair {   // s = s0 + s1 x, r = r0 + r1 x
        double s0, s1, r0, r1;
    };
    auto put = [&](const Pair& a, const Pair& b, double w) {
        out.insert(out.end(), {a.s0, a.s1, a.r0, a.r1, b.s0, b.s1, b.r0, b.r1, w, 0.0});
    };
    // the position w = x of a coordinate pair at offset u: base = x (1 - u)
    auto split = [](double u, bool up) { return up ? Pair{0.0, 1 - u, u, 1 - u} : Pair{u, 1 - u, 0.0, 1 - u}; };
    for (int a = 0; a < n; ++a)
        for (int b = 0; b < n; ++b) {
            const double rho = gx[a], t = gx[b], W = gw[a] * gw[b];
            if (cls == 2) {  // identical: 2 x 2 signs x 2 triangles
                for (int sg = 0; sg < 4; ++sg)
                    for (int tri = 0; tri < 2; ++tri) {
                        const double u1 = tri ? rho * t : rho, u2 = tri ? rho : rho * t;
                        put(split(u1, !(sg & 1)), split(u2, !(sg & 2)), W * (1 - u1) * (1 - u2) * rho);
                    }
            } else if (cls == 1) {  // edge: 2 signs x 3 pyramids
                for (int sg = 0; sg < 2; ++sg)
                    for (int pyr = 0; pyr < 3; ++pyr) {
                        const double u1 = pyr == 0 ? rho : rho * t;
                        const Pair b2 = pyr == 0   ? Pair{rho * t, 0.0, 0.0, rho}
                                        : pyr == 1 ? Pair{rho, 0.0, 0.0, rho}
                                                   : Pair{0.0, rho, rho, 0.0};
                        put(split(u1, !sg), b2, W * (1 - u1) * rho * rho);
                    }
            } else {  // vertex: 4 pyramids, (s1, s2, r1, r2) = rho at one coordinate
                const double W3 = W * rho * rho * rho, q = rho * t;
                put(Pair{rho, 0.0, 0.0, rho}, Pair{q, 0.0, 0.0, rho}, W3);
                put(Pair{q, 0.0, 0.0, rho}, Pair{rho, 0.0, 0.0, rho}, W3);
                put(Pair{0.0, rho, rho, 0.0}, Pair{q, 0.0, 0.0, rho}, W3);
                put(Pair{0.0, rho, q, 0.0}, Pair{0.0, rho, rho, 0.0}, W3);
            }
        }
    return out;
}

}  // namespace

// orders of the GPU rules (see near_classify for the regular ones)
constexpr int NSING_IDENT = 7, NSING_EDGE = 8, NSING_VERTEX = 9;

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
        std::vector<double> r = duffy_blocks(c, ord[c]);
        if ((st = upload(d_rules[c], r.data(), r.size(), nullptr))) return st;
        A.rule[c] = d_rules[c].as<double>();
        A.rule_n[c] = int(r.size() / 10);
        A.rule_ord[c] = ord[c];
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

    // chunks of target elements with a bounded staging buffer
    const int64_t max_slots = std::max<int64_t>(int64_t(1) << 22, 1);  // 4M pairs
    if ((st = alloc(d_stage, size_t(std::min(npairs, max_slots)) * NL * NL * sizeof(double2), nullptr)))
        return st;
    if ((st = alloc(d_list, size_t(std::min(npairs, max_slots)) * sizeof(int), nullptr))) return st;
    A.stage = d_stage.as<double2>();
    const bool hard = op->bc == IGB_HARD;
    int64_t e0 = 0;
    std::vector<int> reg, reg_big, sing;
    const int geo_deg = *std::max_element(g->pg.begin(), g->pg.end());
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
            // the nets are read at the largest geometry degree (2 or 3)
            if (geo_deg <= 2)
                hipLaunchKernelGGL((near_singular<P, HARD, 2>), dim3(unsigned(sing.size())), dim3(NEAR_THREADS), 0, s, A);
            else
                hipLaunchKernelGGL((near_singular<P, HARD, 3>), dim3(unsigned(sing.size())), dim3(NEAR_THREADS), 0, s, A);
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

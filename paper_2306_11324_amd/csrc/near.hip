// Near field of the igafmm library (gfx950): the Galerkin blocks of close and touching
// element pairs by quadrature, gathered into the CSR matrix of the solution space.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "common.h"
#include "near_rules.h"
#include "quadrature_device.h"

namespace igb {

// --------------------------------------------------------------------------
// Near field: regular element pairs (tensor Gauss of order n on both elements)
// --------------------------------------------------------------------------
constexpr int NEAR_THREADS = 256;
constexpr int MASS_ORDER = 6;   // Gauss order per direction of the mass matrix on identical pairs

// Staged places of the near pairs' blocks.  A target element's blocks are stored
// by test function, then source: [a][source][b], the sources ordered by the near
// leaves of the target's leaf and row-major inside each leaf (so a source's place
// follows from its leaf's rank in the list).
struct NearSlots {
    const int64_t* near_ptr;   // [E + 1] first near pair of each target element
    const int* list_ptr;       // [leaves + 1]
    const int* list;           // near leaves of each leaf, sorted
    int d, L, nel1;            // elements per leaf side 2^d, leaf level
};
__device__ __forceinline__ int leaf_index(const NearSlots& S, int patch, int lx, int ly) {
    return (patch << (2 * S.L)) + (ly << S.L) + lx;
}
// position of leaf sl in the near list of leaf tl, -1 if it is not there
__device__ __forceinline__ int near_leaf_rank(const NearSlots& S, int tl, int sl) {
    const int a = S.list_ptr[tl], b = S.list_ptr[tl + 1];
    int lo = a, hi = b;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (S.list[mid] < sl) lo = mid + 1;
        else hi = mid;
    }
    return lo < b && S.list[lo] == sl ? lo - a : -1;
}
// first staged entry of target element e's test function a (nl local functions)
__device__ __forceinline__ int64_t stage_row(const NearSlots& S, int64_t e, int64_t slot0, int nl, int a) {
    const int64_t k = S.near_ptr[e];
    return ((k - slot0) * nl + a * (S.near_ptr[e + 1] - k)) * nl;
}
// place of source element f among the near sources of an element of leaf tl
__device__ __forceinline__ int stage_slot(const NearSlots& S, int tl, int f) {
    const int n2 = S.nel1 * S.nel1, p = f / n2, fy = f % n2 / S.nel1, fx = f % n2 % S.nel1, s1 = (1 << S.d) - 1;
    return (near_leaf_rank(S, tl, leaf_index(S, p, fx >> S.d, fy >> S.d)) << (2 * S.d)) + ((fy & s1) << S.d) + (fx & s1);
}
__device__ __forceinline__ int leaf_of(const NearSlots& S, int64_t e) {
    const int n2 = S.nel1 * S.nel1, p = int(e / n2), r = int(e % n2);
    return leaf_index(S, p, r % S.nel1 >> S.d, r / S.nel1 >> S.d);
}

struct NearArgs {
    const double* bez;
    const int* pg;
    const double* C1;
    const double* gl;        // [NGMAX+1][2][NGMAX]: Gauss nodes / weights on [0,1] per order
    NearSlots slots;
    const int* leaf_src;           // near source elements of each leaf, sorted
    const int64_t* leaf_src_ptr;   // [leaves + 1]
    const unsigned short* code;    // near pair -> Gauss orders, 0 for a touching pair
    const NearTouch* touch;        // touching pairs handled by this launch
    int64_t slot0;           // first staged pair
    double2* stage;          // [pairs][nloc*nloc], order: NearSlots
    int nel1;
    int seg;                 // pairs per workgroup of the regular kernel, at most REG_SEG
    double kappa;
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

// --------------------------------------------------------------------------
// Near field: regular element pairs, tensor Gauss rules of orders (nu, nv) on
// each element (the orders may differ between the two elements and between
// directions).
//
// One wave takes a target element and a segment of its pairs, one rule at a
// time: the test points once, then batches of source elements with one source
// point per lane, and then the batch's points 16 at a time.  Lane (g, li)
// evaluates the kernel at source point li and test points 4 t + g, which is the A
// operand of the first product T[j][a] = sum_i k(x_i, y_j) w phi_a(x_i) on the
// fp64 matrix cores; its result, rows 4 r + g in register r, is the B operand of
// the second product B[b][a] = sum_j w phi_b(y_j) T[j][a] as it stands, so no
// value passes through LDS between evaluation and the finished block.  Test
// points are padded to 4 per element and source points to 4 per source (weight
// 0, so their values do not matter).
// (Sound-hard: the curl parts c_a . c_b as three more components with the kernel g.)
// One wave per workgroup, so that no wave waits for another at the many small
// rules of an element (16-20 of them, most with a few pairs).  Bound by fp64
// issue: about 80 VALU instructions per point pair, 125 per source element to
// place its points, and the padded matrix products, which run on the same fp64
// units.  Level-5 sphere, p = 2, leaf depth 3, 17.6 million pairs: 128 -> 44 ms
// (before: a workgroup per pair, values and products through LDS); level-5 hard
// star, 5.3 million pairs: 73 -> 37 ms.  Segments of 1024 pairs left a quarter of
// the CU time idle at the end of a launch (52 and 39 ms), of 128 set up their
// rules too often (48).
// --------------------------------------------------------------------------
typedef double f64x4 __attribute__((ext_vector_type(4)));

// points of the larger of a regular pair's two rules
__device__ __forceinline__ int regular_points(int code) {
    const int nx = (code & 15) * ((code >> 4) & 15), ny = ((code >> 8) & 15) * (code >> 12);
    return nx > ny ? nx : ny;
}
constexpr int REG_SEG = 256;           // pairs per workgroup at most
constexpr int REG_SEG_MIN = 16;        // and at least (a batch's sources), where there are few
constexpr int REG_WAVES = 2048;        // waves that fill the device: 2 per SIMD

// point data of a regular rule: g[0..6] = x, n~, |n~|; sound-hard also F_s, F_t
template <bool HARD>
__device__ __forceinline__ void surface_point(const ElemRef& R, double s, double t, double* g) {
    GeoPt G;
    if (R.pu == 2 && R.pv == 2) {
        // all 9 control points in flight together
        const double2* H = reinterpret_cast<const double2*>(R.bez);
        double2 h[3][3][2];
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int c = 0; c < 2; ++c) h[j][i][c] = H[(j * (PGMAX + 1) + i) * 2 + c];
        double bu[4], du[4], bv[4], dv[4];
        bernstein(2, s, bu, du);
        bernstein(2, t, bv, dv);
        double p[4], ps[4], pt[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            double v = 0, vs = 0, vt = 0;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                double r = 0, rs = 0;
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const double x = c & 1 ? h[j][i][c >> 1].y : h[j][i][c >> 1].x;
                    r = fma(bu[i], x, r);
                    rs = fma(du[i], x, rs);
                }
                v = fma(bv[j], r, v);
                vs = fma(bv[j], rs, vs);
                vt = fma(dv[j], r, vt);
            }
            p[c] = v;
            ps[c] = vs;
            pt[c] = vt;
        }
        const double iw = rcp_fast(p[3]);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            G.x[c] = p[c] * iw;
            G.fs[c] = (ps[c] - G.x[c] * ps[3]) * iw;
            G.ft[c] = (pt[c] - G.x[c] * pt[3]) * iw;
        }
    } else {
        eval_geo(R.bez, R.pu, R.pv, s, t, G);
    }
    double nt[3];
    cross3(G.fs, G.ft, nt);
    const double n2 = nt[0] * nt[0] + nt[1] * nt[1] + nt[2] * nt[2];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        g[c] = G.x[c];
        g[3 + c] = nt[c];
        if (HARD) {
            g[7 + c] = G.fs[c];
            g[10 + c] = G.ft[c];
        }
    }
    g[6] = n2 * rsqrt_fast(n2);
}

template <int P, bool HARD, int MX>
__global__ __launch_bounds__(64, 2) void near_regular(NearArgs A, int e0) {
    constexpr int P1 = P + 1, NL = P1 * P1, NV = HARD ? 4 : 1, NG = HARD ? 13 : 7, ND = HARD ? 2 * P1 : P1;
    constexpr int YC = regular_batch_points(MX);   // source points per batch (at least one source)
    static_assert(MX % 4 == 0 && MX <= REG_POINTS_MAX, "padded points of a rule");
    __shared__ unsigned short code[REG_SEG], list[REG_SEG];
    __shared__ double xg[MX][NG], yg[YC][NG];
    __shared__ double px[HARD ? 1 : MX][NL], py[HARD ? 1 : YC][NL];   // sound-soft: w phi at the test and source points
    __shared__ double bx[2 * REG_ORDER_MAX][ND];          // 1-D basis values (then derivatives) at the test points: u, v
    __shared__ double by[REG_BASIS_ROWS][ND];             // the same per source of a batch: [source][u, v]
    __shared__ int lsrc[REG_BATCH_MAX], lslot[REG_BATCH_MAX];
    const int e = e0 + blockIdx.x, lane = threadIdx.x, li = lane & 15, g = lane >> 4;
    const int lc = min(li, NL - 1), lu = lc % P1, lv = lc / P1;   // basis index of this lane (past NL: not read)
    const int64_t kb = A.slots.near_ptr[e] + int64_t(blockIdx.y) * A.seg;
    const int np = int(min(int64_t(A.seg), A.slots.near_ptr[e + 1] - kb));
    if (np <= 0) return;
    const int tl = leaf_of(A.slots, e);
    const int* src = A.leaf_src + A.leaf_src_ptr[tl] + int64_t(blockIdx.y) * A.seg;   // sources of the segment's pairs
    const ElemRef Re = elem_ref(A.bez, A.pg, A.nel1, e);
    constexpr int NONE = 0xffff;   // (orders are at most 12: no rule has this code)
    int next = NONE;
    for (int k = lane; k < np; k += 64) {
        const int kd = A.code[kb + k];
        const bool mine = kd != 0 && (regular_points(kd) <= REG_POINTS_SMALL) == (MX == REG_POINTS_SMALL);
        const int c = mine ? kd : NONE;
        code[k] = (unsigned short)c;
        next = min(next, c);
    }
    // 1-D basis of an element at the nodes of order n along one direction, times the weight
    auto basis = [&](int n, int r, const double* C, double* o) {
        const double* gl = A.gl + n * 2 * NGMAX;
        double b[P1], db[P1];
        eval_basis1<P>(C, gl[r], b, db);
#pragma unroll
        for (int a = 0; a < P1; ++a) {
            o[a] = gl[NGMAX + r] * b[a];
            if (HARD) o[ND - P1 + a] = gl[NGMAX + r] * db[a];
        }
    };
    // component v of the weighted test functions at a point (u and v factors bu, bv, geometry p):
    // phi, then the curl d_s phi F_t - d_t phi F_s
    auto comp = [&](int v, const double* bu, const double* bv, const double* p) {
        if (v == 0) return bu[lu] * bv[lv];
        return bu[ND - P1 + lu] * bv[lv] * p[9 + v] - bu[lu] * bv[ND - P1 + lv] * p[6 + v];
    };
    for (;;) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) next = min(next, __shfl_xor(next, o, 64));
        const int cur = next;
        if (cur == NONE) break;
        const int nxu = cur & 15, nxv = (cur >> 4) & 15, nyu = (cur >> 8) & 15, nyv = cur >> 12;
        const int nx = nxu * nxv, ny = nyu * nyv, nx4 = regular_padded(nx), ny4 = regular_padded(ny), n1 = nyu + nyv;
        const double *gxu = A.gl + nxu * 2 * NGMAX, *gxv = A.gl + nxv * 2 * NGMAX;
        const double *gyu = A.gl + nyu * 2 * NGMAX, *gyv = A.gl + nyv * 2 * NGMAX;
        __syncthreads();   // the rule before is done with the LDS
        // the rule's pairs in order, and the next rule
        int nsrc = 0;
        next = NONE;
        for (int k0 = 0; k0 < np; k0 += 64) {
            const int c = k0 + lane < np ? code[k0 + lane] : NONE;
            const unsigned long long m = __ballot(c == cur);
            if (c == cur) list[nsrc + __popcll(m & ((1ull << lane) - 1))] = (unsigned short)(k0 + lane);
            if (c > cur) next = min(next, c);
            nsrc += __popcll(m);
        }
        for (int i = lane; i < nx4; i += 64) {
            const int j = i < nx ? i : 0;
            surface_point<HARD>(Re, gxu[j % nxu], gxv[j / nxu], xg[i]);
        }
        for (int r = lane; r < nxu + nxv; r += 64) {
            const bool u = r < nxu;
            basis(u ? nxu : nxv, u ? r : r - nxu, A.C1 + (u ? Re.ex : Re.ey) * P1 * P1, bx[r]);
        }
        __syncthreads();
        if (!HARD)
            for (int t = lane; t < nx4 * NL; t += 64) {
                const int i = t / NL, a = t % NL;
                px[i][a] = i < nx ? bx[i % nxu][a % P1] * bx[nxu + i / nxu][a / P1] : 0.0;
            }
        const int nbmax = regular_batch(MX, nyu, nyv);
        const int invx = (65536 + nxu - 1) / nxu, invy = (65536 + nyu - 1) / nyu;   // i / n = i * inv >> 16 for i < 144
        for (int s0 = 0; s0 < nsrc; s0 += nbmax) {
            const int nb = min(nbmax, nsrc - s0), je = nb * ny4;
            __syncthreads();   // the batch before is read
            if (lane < nb) {
                const int f = src[list[s0 + lane]];
                lsrc[lane] = f;
                lslot[lane] = stage_slot(A.slots, tl, f);
            }
            __syncthreads();
            for (int t = lane; t < je; t += 64) {
                const int q = t / ny4, j = t - q * ny4, jj = j < ny ? j : 0, jv = jj * invy >> 16;
                surface_point<HARD>(elem_ref(A.bez, A.pg, A.nel1, lsrc[q]), gyu[jj - jv * nyu], gyv[jv], yg[t]);
            }
            for (int t = lane; t < nb * n1; t += 64) {
                const int q = t / n1, r = t - q * n1;
                const bool u = r < nyu;
                const ElemRef Rf = elem_ref(A.bez, A.pg, A.nel1, lsrc[q]);
                basis(u ? nyu : nyv, u ? r : r - nyu, A.C1 + (u ? Rf.ex : Rf.ey) * P1 * P1, by[t]);
            }
            __syncthreads();
            if constexpr (!HARD) {
                for (int t = lane; t < je; t += 64) {
                    const int q = t / ny4, j = t - q * ny4, jj = j < ny ? j : 0, jv = jj * invy >> 16;
                    const double *pu = by[q * n1 + jj - jv * nyu], *pv = by[q * n1 + nyu + jv];
                    const double on = j < ny ? 1.0 : 0.0;
#pragma unroll
                    for (int b = 0; b < NL; ++b) py[t][b] = on * (pu[b % P1] * pv[b / P1]);
                }
                __syncthreads();
            }
            f64x4 cr = {0, 0, 0, 0}, ci = {0, 0, 0, 0};
            int q = 0, qend = ny4;   // current source of the batch, its end
            auto store = [&]() {
                double2* o = A.stage + stage_row(A.slots, e, A.slot0, NL, lc) + int64_t(lslot[q]) * NL;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (li < NL && g + 4 * r < NL) o[g + 4 * r] = make_double2(cr[r], ci[r]);
            };
            for (int jt = 0; jt < je; jt += 16) {
                const int J = min(jt + li, je - 1);
                double Y[7];
#pragma unroll
                for (int c = 0; c < 7; ++c) Y[c] = yg[J][c];
                f64x4 tr[NV], ti[NV];
#pragma unroll
                for (int v = 0; v < NV; ++v) tr[v] = ti[v] = f64x4{0, 0, 0, 0};
                for (int t = 0; t < nx4; t += 4) {
                    const double* X = xg[t + g];
                    const KVal kv = kernel_pair<HARD>(X, X + 3, X[6], Y, Y + 3, Y[6], A.kappa, A.mix, A.hmix);
                    if constexpr (!HARD) {
                        const double ph = px[t + g][lc];
                        tr[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(kv.s.x, ph, tr[0], 0, 0, 0);
                        ti[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(kv.s.y, ph, ti[0], 0, 0, 0);
                    } else {
                        const int i = t + g, iv = i * invx >> 16;
                        const double *pu = bx[i < nx ? i - iv * nxu : 0], *pv = bx[i < nx ? nxu + iv : 0];
                        const double on = i < nx ? 1.0 : 0.0;
#pragma unroll
                        for (int v = 0; v < NV; ++v) {
                            const double ph = on * comp(v, pu, pv, X);
                            const double2 k = v == 0 ? kv.s : kv.g;
                            tr[v] = __builtin_amdgcn_mfma_f64_16x16x4f64(k.x, ph, tr[v], 0, 0, 0);
                            ti[v] = __builtin_amdgcn_mfma_f64_16x16x4f64(k.y, ph, ti[v], 0, 0, 0);
                        }
                    }
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int jk = jt + 4 * r;
                    if (jk >= je) break;
                    if (jk == qend) {   // the source before is complete
                        store();
                        cr = ci = f64x4{0, 0, 0, 0};
                        ++q;
                        qend += ny4;
                    }
                    if constexpr (!HARD) {
                        const double ph = py[jk + g][lc];
                        cr = __builtin_amdgcn_mfma_f64_16x16x4f64(ph, tr[0][r], cr, 0, 0, 0);
                        ci = __builtin_amdgcn_mfma_f64_16x16x4f64(ph, ti[0][r], ci, 0, 0, 0);
                        continue;
                    }
                    const int j = jk + g - (qend - ny4), jv = j * invy >> 16;
                    const bool in = j < ny;
                    const double *pu = by[q * n1 + (in ? j - jv * nyu : 0)], *pv = by[q * n1 + nyu + (in ? jv : 0)];
                    const double on = in ? 1.0 : 0.0;
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        const double ph = on * comp(v, pu, pv, yg[jk + g]);
                        cr = __builtin_amdgcn_mfma_f64_16x16x4f64(ph, tr[v][r], cr, 0, 0, 0);
                        ci = __builtin_amdgcn_mfma_f64_16x16x4f64(ph, ti[v][r], ci, 0, 0, 0);
                    }
                }
            }
            store();
        }
    }
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
// entry (k, i) of the degree elevation from p to q >= p: b^q_k = sum_i E(k, i) b^p_i
__device__ __forceinline__ double elevation(int p, int q, int k, int i) {
    constexpr double C[4][4] = {{1, 0, 0, 0}, {1, 1, 0, 0}, {1, 2, 1, 0}, {1, 3, 3, 1}};
    const int r = k - i;
    return r < 0 || r > q - p ? 0.0 : C[p][i] * C[q - p][r] / C[q][k];
}

// P: spline degree, G >= the geometry degree of every element (lower degrees are
// elevated as the net is read)
template <int P, bool HARD, int G>
__global__ __launch_bounds__(NEAR_THREADS, !HARD && P <= 2 && G == 2 ? 2 : 1) void near_singular(NearArgs A) {
    constexpr int P1 = P + 1, NL = P1 * P1, G1 = G + 1, NW = NEAR_THREADS / 64;
    constexpr int NT = HARD ? 4 : 1;   // factorised terms with their own outer factor
    // terms summed per walk along a line (degree 3: two walks of two, within the registers)
    constexpr int TW = HARD && P == 3 ? 2 : NT;
    __shared__ double net[2][G1][G1][4];      // [x, y][dim 1][dim 2][homogeneous]
    __shared__ double ext[2][2][P1][P1];      // [x, y][dim][B-spline][Bernstein]
    __shared__ double2 Tb[NW][64][NL];        // a chunk's inner sums, one term at a time
    __shared__ double Qb[NW][64][NL];         // and its outer factors
    __shared__ double2 Mb[NL][NL], Rb[NL][NL];
    __shared__ double mw[MASS_ORDER * MASS_ORDER], mb[MASS_ORDER * MASS_ORDER * 2 * P1];   // mass matrix points
    double2* red = &Tb[0][0][0];              // [NW][NL][NL] after the loop
    static_assert(sizeof(double2) * NW * NL * NL <= sizeof(Tb), "the waves' sums fit");

    const NearTouch pair = A.touch[blockIdx.x];
    const int kind = pair.kind;
    const int cls = kind & 15;
    const int ri = cls == 4 ? 2 : cls == 2 ? 1 : 0;
    const double* rule = A.rule[ri];
    const int n = A.rule_ord[ri], nlines = A.rule_n[ri] * n;
    const double* gx = A.gl + n * 2 * NGMAX;
    const double* gw = gx + NGMAX;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, g = lane >> 4;
    const int code[2] = {(kind >> 16) & 7, (kind >> 20) & 7};
    const ElemRef R[2] = {elem_ref(A.bez, A.pg, A.nel1, pair.e), elem_ref(A.bez, A.pg, A.nel1, pair.f)};

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
        for (int t0 = 0; t0 < NT; t0 += TW) {
        double2 T[TW][P1][P1];
#pragma unroll
        for (int t = 0; t < TW; ++t)
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
            const double2 Gw = HARD ? cscale(kv.g, wa * sxy) : make_double2(0, 0);
            // T[t][i][k] += K f_i(s1) h_k(r1), f and h Bernstein values or derivatives
            auto add = [&](double2(&Tt)[P1][P1], double2 K, const double* f, const double* h) {
#pragma unroll
                for (int i = 0; i < P1; ++i) {
                    const double2 u = cscale(K, f[i]);
#pragma unroll
                    for (int k = 0; k < P1; ++k) {
                        Tt[i][k].x = fma(u.x, h[k], Tt[i][k].x);
                        Tt[i][k].y = fma(u.y, h[k], Tt[i][k].y);
                    }
                }
            };
            auto dot = [](const double* a, const double* b) { return a[0] * b[0] + a[1] * b[1] + a[2] * b[2]; };
            if (t0 == 0) {
                add(T[0], S, bx, by);
                if constexpr (HARD) {
                    add(T[0], cscale(Gw, dot(F2[0], F2[1])), dbx, dby);
                    add(T[1], cscale(Gw, -dot(F2[0], F1[1])), dbx, by);
                }
            }
            if constexpr (HARD) {
                if (TW == NT || t0 > 0) {
                    add(T[TW - 2], cscale(Gw, -dot(F1[0], F2[1])), bx, dby);
                    add(T[TW - 1], cscale(Gw, dot(F1[0], F1[1])), bx, by);
                }
            }
        }
        // outer factors (weighted): b_j b_l, and sound-hard b_j d_l, d_j b_l, d_j d_l
        double bx[4], dbx[4], by[4], dby[4];
        bernstein(P, s2, bx, dbx);
        bernstein(P, r2, by, dby);
#pragma unroll
        for (int tt = 0; tt < TW; ++tt) {
            const int t = t0 + tt;
            wave_lds_sync();   // the previous term's operands are read
#pragma unroll
            for (int i = 0; i < P1; ++i)
#pragma unroll
                for (int k = 0; k < P1; ++k) {
                    Tb[wave][lane][i * P1 + k] = T[tt][i][k];
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
        // (identical pairs carry no symmetry: the net is in element coordinates)
        double bu[4], du[4], bv[4], dv[4], p0[4], p1[4], p2[4];
        bernstein(G, ss, bu, du);
        bernstein(G, tt, bv, dv);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            p0[c] = p1[c] = p2[c] = 0;
#pragma unroll
            for (int i = 0; i < G1; ++i)
#pragma unroll
                for (int j = 0; j < G1; ++j) {
                    const double h = net[0][i][j][c];
                    p0[c] = fma(bu[i] * bv[j], h, p0[c]);
                    p1[c] = fma(du[i] * bv[j], h, p1[c]);
                    p2[c] = fma(bu[i] * dv[j], h, p2[c]);
                }
        }
        const double iw = 1.0 / p0[3];
        double fs[3], ft[3], nt[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            fs[c] = (p1[c] - p0[c] * iw * p1[3]) * iw;
            ft[c] = (p2[c] - p0[c] * iw * p2[3]) * iw;
        }
        cross3(fs, ft, nt);
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
        const int slot = stage_slot(A.slots, leaf_of(A.slots, pair.e), pair.f);
        A.stage[stage_row(A.slots, pair.e, A.slot0, NL, oa) + int64_t(slot) * NL + ob] = s;
    }
}

// --------------------------------------------------------------------------
// Near field: deterministic gather of the staged element blocks into the CSR
// values of the solution space.  One workgroup per row; each nonzero sums its
// contributions in a fixed order (representatives, leaves and elements of the
// row, source elements).  A source element's staged place follows from its
// leaf's place in the target leaf's near list (stage_slot), so a nonzero searches
// that list once per target and source leaf instead of the element's pairs once
// per element pair, and then has the (p+1)^2 loads of a target element in
// flight together.  Bound by the staged blocks' traffic (16 (p+1)^4 bytes per
// near pair, written and read once).  Level-5 sphere, leaf depth 3, p = 2 (23 GB
// of blocks): 39 -> 11 ms.
// --------------------------------------------------------------------------
struct CsrArgs {
    const int64_t* row_ptr;
    const int64_t* row_coff;     // first entry of the row's column list in col
    const int* col;
    double2* val;
    NearSlots slots;
    const double2* stage;
    int64_t slot0;
    int64_t e_lo, e_hi;          // target elements whose pairs are staged
    const int* s0_ptr;           // null for S^2 (soft)
    const int* s0_reps;
    int64_t row0;
    int nel1, k;
};

template <int P>
__global__ __launch_bounds__(256) void near_gather_csr(CsrArgs A) {
    constexpr int P1 = P + 1, NL = P1 * P1;
    const int64_t row = A.row0 + blockIdx.x;
    const int64_t beg = A.row_ptr[row], end = A.row_ptr[row + 1];
    const int* col = A.col + A.row_coff[row] - beg;
    const int kk = A.k * A.k, d = A.slots.d, s1 = (1 << d) - 1, n1 = A.nel1 - 1;
    const int r0 = A.s0_ptr ? A.s0_ptr[row] : int(row);
    const int r1 = A.s0_ptr ? A.s0_ptr[row + 1] : int(row) + 1;
    for (int64_t idx = beg + threadIdx.x; idx < end; idx += blockDim.x) {
        const int colv = col[idx];
        const int c0 = A.s0_ptr ? A.s0_ptr[colv] : colv;
        const int c1 = A.s0_ptr ? A.s0_ptr[colv + 1] : colv + 1;
        double2 acc = make_double2(0, 0);
        for (int ri = r0; ri < r1; ++ri) {
            const int i = A.s0_ptr ? A.s0_reps[ri] : ri;
            const int pj = i / kk, iv = i % kk / A.k, iu = i % kk % A.k;
            const int ey0 = max(0, iv - P), ey1 = min(iv, n1), ex0 = max(0, iu - P), ex1 = min(iu, n1);
            for (int ly = ey0 >> d; ly <= ey1 >> d; ++ly)
                for (int lx = ex0 >> d; lx <= ex1 >> d; ++lx) {
                    const int tl = leaf_index(A.slots, pj, lx, ly);
                    for (int ci = c0; ci < c1; ++ci) {
                        const int j = A.s0_ptr ? A.s0_reps[ci] : ci;
                        const int qj = j / kk, jv = j % kk / A.k, ju = j % kk % A.k;
                        // staged places of the source elements jv - dy, ju - dx relative to the
                        // target element's blocks (-1: not a near source)
                        int off[NL], lf[P1], lq[P1];
#pragma unroll
                        for (int dx = 0; dx < P1; ++dx) lf[dx] = -1;
#pragma unroll
                        for (int dy = 0; dy < P1; ++dy)
#pragma unroll
                            for (int dx = 0; dx < P1; ++dx) {
                                const int fy = jv - dy, fx = ju - dx;
                                const bool in = fy >= 0 && fy <= n1 && fx >= 0 && fx <= n1;
                                const int sl = in ? leaf_index(A.slots, qj, fx >> d, fy >> d) : -1;
                                if (sl != lf[dx]) {
                                    lf[dx] = sl;
                                    lq[dx] = dx > 0 && sl == lf[dx - 1] ? lq[dx - 1] : near_leaf_rank(A.slots, tl, sl);
                                }
                                off[dy * P1 + dx] =
                                    in && lq[dx] >= 0
                                        ? ((lq[dx] << (2 * d)) + ((fy & s1) << d) + (fx & s1)) * NL + dy * P1 + dx
                                        : -1;
                            }
                        for (int ey = max(ey0, ly << d); ey <= min(ey1, (ly << d) + s1); ++ey)
                            for (int ex = max(ex0, lx << d); ex <= min(ex1, (lx << d) + s1); ++ex) {
                                const int64_t e = (int64_t(pj) * A.nel1 + ey) * A.nel1 + ex;
                                if (e < A.e_lo || e >= A.e_hi) continue;
                                const int a = (iv - ey) * P1 + (iu - ex);
                                const double2* blk = A.stage + stage_row(A.slots, e, A.slot0, NL, a);
                                double2 v[NL];
#pragma unroll
                                for (int t = 0; t < NL; ++t)
                                    v[t] = off[t] >= 0 ? blk[off[t]] : make_double2(0, 0);
#pragma unroll
                                for (int t = 0; t < NL; ++t) acc = cadd(acc, v[t]);
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
    DevBuf d_code, d_leaf_src, d_leaf_src_ptr, d_gl, d_rules[3], d_touch, d_stage;
    if ((st = upload(d_code, op->near_code.data(), op->near_code.size(), nullptr)) ||
        (st = upload(d_leaf_src, op->leaf_src.data(), op->leaf_src.size(), nullptr)) ||
        (st = upload(d_leaf_src_ptr, op->leaf_src_ptr.data(), op->leaf_src_ptr.size(), nullptr)))
        return st;
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
    if ((st = upload(op->d_rowptr, op->row_ptr.data(), op->row_ptr.size(), acct))) return st;
    if ((st = upload(op->d_dcol, op->near_dcol.data(), op->near_dcol.size(), acct))) return st;
    if ((st = upload(op->d_row_coff, op->row_coff.data(), op->row_coff.size(), acct))) return st;
    if ((st = upload(op->d_near_wgs, op->near_wgs.data(), op->near_wgs.size(), acct))) return st;
    if ((st = upload(op->d_near_grp_rows, op->near_grp_rows.data(), op->near_grp_rows.size(), acct))) return st;
    if ((st = alloc(op->d_val, op->nnz * sizeof(double2), acct))) return st;
    IGB_HIP(hipMemsetAsync(op->d_val.ptr, 0, op->nnz * sizeof(double2), s));

    std::vector<int> list_ptr(op->near_leaf.size() + 1, 0), list;
    for (size_t i = 0; i < op->near_leaf.size(); ++i) {
        list.insert(list.end(), op->near_leaf[i].begin(), op->near_leaf[i].end());
        list_ptr[i + 1] = int(list.size());
    }
    DevBuf d_list_ptr, d_list;
    if ((st = upload(d_list_ptr, list_ptr.data(), list_ptr.size(), nullptr)) ||
        (st = upload(d_list, list.data(), list.size(), nullptr)))
        return st;
    const NearSlots slots{op->d_near_ptr.as<int64_t>(), d_list_ptr.as<int>(), d_list.as<int>(), op->d, op->L, g->nel1};

    A.bez = g->d_bez.as<double>();
    A.pg = g->d_pg.as<int>();
    A.C1 = g->d_C1.as<double>();
    A.gl = d_gl.as<double>();
    A.slots = slots;
    A.leaf_src = d_leaf_src.as<int>();
    A.leaf_src_ptr = d_leaf_src_ptr.as<int64_t>();
    A.code = d_code.as<unsigned short>();
    A.nel1 = g->nel1;
    A.kappa = op->kappa;
    A.mix = op->mix;
    A.hmix = op->hmix;
    A.cm = op->cm;

    // chunks of target elements with a bounded staging buffer
    const int64_t max_slots = std::max<int64_t>(int64_t(1) << 22, 1);  // 4M pairs
    if ((st = alloc(d_stage, size_t(std::min(npairs, max_slots)) * NL * NL * sizeof(double2), nullptr)))
        return st;
    if ((st = upload(d_touch, op->near_touch.data(), op->near_touch.size(), nullptr))) return st;
    A.stage = d_stage.as<double2>();
    const bool hard = op->bc == IGB_HARD;
    int64_t e0 = 0;
    const int geo_deg = *std::max_element(g->pg.begin(), g->pg.end());
    while (e0 < E) {
        int64_t e1 = e0;
        while (e1 < E && op->near_ptr[e1 + 1] - op->near_ptr[e0] <= max_slots) ++e1;
        if (e1 == e0) {
            set_error("assemble_nearfield: one element has more near pairs than the staging buffer");
            return IGB_ERR_UNSUPPORTED;
        }
        const int64_t k0 = op->near_ptr[e0];
        A.slot0 = k0;
        // regular pairs, a workgroup per target element and segment of its pairs
        int64_t longest = 0;
        for (int64_t e = e0; e < e1; ++e) longest = std::max(longest, op->near_ptr[e + 1] - op->near_ptr[e]);
        // (few elements: shorter segments until the waves fill the device, as a wave walks
        // its pairs one batch after another; a pair's block does not depend on it)
        A.seg = REG_SEG;
        while (A.seg > REG_SEG_MIN && (e1 - e0) * ((longest + A.seg - 1) / A.seg) < REG_WAVES) A.seg /= 2;
        const dim3 rgrid(unsigned(e1 - e0), unsigned((longest + A.seg - 1) / A.seg));
        hipLaunchKernelGGL((near_regular<P, HARD, REG_POINTS_SMALL>), rgrid, dim3(64), 0, s, A, int(e0));
        if (op->near_points_max > REG_POINTS_SMALL)
            hipLaunchKernelGGL((near_regular<P, HARD, REG_POINTS_MAX>), rgrid, dim3(64), 0, s, A, int(e0));
        IGB_HIP(hipGetLastError());
        // touching pairs (the nets are read at the largest geometry degree, 2 or 3)
        const int64_t t0 = op->near_touch_ptr[e0], nt = op->near_touch_ptr[e1] - t0;
        A.touch = d_touch.as<NearTouch>() + t0;
        if (nt > 0 && geo_deg <= 2)
            hipLaunchKernelGGL((near_singular<P, HARD, 2>), dim3(unsigned(nt)), dim3(NEAR_THREADS), 0, s, A);
        else if (nt > 0)
            hipLaunchKernelGGL((near_singular<P, HARD, 3>), dim3(unsigned(nt)), dim3(NEAR_THREADS), 0, s, A);
        IGB_HIP(hipGetLastError());
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
        C.row_coff = op->d_row_coff.as<int64_t>();
        C.col = op->d_dcol.as<int>();
        C.val = op->d_val.as<double2>();
        C.slots = slots;
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

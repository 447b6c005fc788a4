"""Near-field quadrature kernels at every spline degree and geometry degree.

The touching-pair kernel reads the control nets at degree 2 or 3 (lower degrees
elevated) and contracts in Bernstein form: the matrix must not depend on the
degree a patch is written in, and must equal the dense oracle's.
"""
from math import comb

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2306_11324_amd import inputs as I

DEGREES = [("soft", 0), ("soft", 1), ("soft", 2), ("soft", 3), ("hard", 1), ("hard", 2), ("hard", 3)]


def B():
    from paper_2306_11324_amd import binding
    return binding


def elevated(patches, q):
    """The same single-span patches written with degree q in both directions."""
    out = []
    for pt in patches:
        hom = np.concatenate([pt.cpw[..., :3] * pt.cpw[..., 3:], pt.cpw[..., 3:]], axis=-1)
        E = [np.array([[comb(d, i) * comb(q - d, k - i) / comb(q, k) if 0 <= k - i <= q - d else 0.0
                        for i in range(d + 1)] for k in range(q + 1)]) for d in (pt.deg_u, pt.deg_v)]
        h = np.einsum("lj,ki,jic->lkc", E[1], E[0], hom)
        kn = np.array([0.0] * (q + 1) + [1.0] * (q + 1))
        out.append(I.Patch(q, q, kn, kn.copy(), np.concatenate([h[..., :3] / h[..., 3:], h[..., 3:]], axis=-1)))
    return out


def cube():
    """Six bilinear patches."""
    kn = np.array([0.0, 0.0, 1.0, 1.0])
    out = []
    for n, e1, e2 in I.CUBE_FACES:
        n, e1, e2 = (np.array(a, dtype=np.float64) for a in (n, e1, e2))
        net = np.ones((2, 2, 4))
        for j in range(2):
            for i in range(2):
                net[j, i, :3] = n + (2 * i - 1) * e1 + (2 * j - 1) * e2
        out.append(I.Patch(1, 1, kn.copy(), kn.copy(), net))
    return out


def near_matrix(patches, m, p, bc, quad_extra=0):
    b = B()
    ctx = b.Context(0)
    geo = b.Geometry(ctx, patches, m, p)
    # nothing admissible: the near field is the whole matrix
    op = b.Operator(ctx, geo, kappa=1.5, bc=b.SOFT if bc == "soft" else b.HARD, q=2, eta_adm=1e6, leaf_depth=1,
                    quad_extra=quad_extra)
    rp, col, val = op.near_csr()
    assert op.info.far_pairs == 0
    return rp, col, val


@pytest.mark.parametrize("bc,p", DEGREES)
@pytest.mark.parametrize("surface", ["sphere", "cube"])
def test_matrix_does_not_depend_on_the_geometry_degree(surface, bc, p):
    # rounding only: positions are rounded at 1e-16, the touching rules' innermost
    # points lie 1e-2 apart where the normal component is known to 1e-12 of the
    # kernel's value, and they carry a small share of the sum: 1e-11 of the largest entry
    base = I.sphere_patches() if surface == "sphere" else cube()
    q = 3 if surface == "sphere" else 2
    rp, col, val = near_matrix(base, 2, p, bc)
    rp2, col2, val2 = near_matrix(elevated(base, q), 2, p, bc)
    assert np.array_equal(rp, rp2) and np.array_equal(col, col2)
    assert np.abs(val - val2).max() <= 1e-11 * np.abs(val).max()


@pytest.mark.parametrize("bc,p", [("soft", 0), ("soft", 3), ("hard", 3)])
def test_matrix_row_matches_dense_oracle(bc, p):
    # the row of a basis function inside the first patch; independent rules on the
    # coarse sphere (24 elements), each accurate to about 1e-7 of the largest entry there
    from oracle import galerkin as G
    pts = I.sphere_patches()
    rp, col, val = near_matrix(pts, 1, p, bc, quad_extra=3)
    ref = G.DenseBEM(pts, p=p, m=1, kappa=1.5, bc=bc, workers=1)
    k = 2 + p
    row = (k // 2) * k + k // 2
    if bc == "hard":
        row = int(ref.disc.s0_map()[0][row])
    a = np.zeros(len(rp) - 1, dtype=np.complex128)
    a[col[rp[row]:rp[row + 1]]] = val[rp[row]:rp[row + 1]]
    r = ref.rows(np.array([row]))[0]
    assert np.abs(a - r).max() <= 1e-6 * np.abs(r).max()

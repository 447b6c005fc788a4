"""Near field of a bar at quad_extra = -2, where the regular kernel's batches of source
elements are bound by their 1-D basis rows: the matrix entries of element pairs that
do not touch, against the oracle's blocks on the same tensor rules."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from test_near_batches import bar, full_batches


@pytest.mark.parametrize("bc,p", [("soft", 0), ("soft", 1), ("soft", 2), ("soft", 3),
                                  ("hard", 1), ("hard", 2), ("hard", 3)])
def test_entries_of_regular_pairs(bc, p):
    from oracle import galerkin as G
    from oracle import quadrature as qd
    from paper_2306_11324_amd import binding as B
    patches, kappa = bar(), 1.0
    ctx = B.Context(0)
    op = B.Operator(ctx, B.Geometry(ctx, patches, 3, p), kappa=kappa, bc=B.SOFT if bc == "soft" else B.HARD, q=2,
                    eta_adm=1e6, leaf_depth=1, quad_extra=-2)
    assert op.info.far_pairs == 0
    ptr, src, kind = op.near_pairs()
    rp, col, val = op.near_csr()
    ref = G.DenseBEM(patches, p=p, m=3, kappa=kappa, bc=bc, workers=1)
    disc, ops = ref.disc, ref.ops
    c0, c1 = (1.0, -1j * ref.eta) if bc == "soft" else (-1.0, -1j * ref.eta)   # of K* and V; of K and W
    fold = np.arange(disc.n2) if bc == "soft" else disc.s0_map()[0]
    full = full_batches(ptr, kind)
    checked = 0
    for e0 in (full[0], full[-1]):
        row = int(fold[disc.el_dofs[e0, 0]])
        want = np.zeros(op.n, dtype=np.complex128)
        known = np.ones(op.n, dtype=bool)
        for e in np.nonzero((fold[disc.el_dofs] == row).any(axis=1))[0]:
            f, k = src[ptr[e]:ptr[e + 1]], kind[ptr[e]:ptr[e + 1]]
            known[fold[disc.el_dofs[f[(k & 15) != 0]]]] = False
            for code in np.unique(k[(k & 15) == 0]):
                fs = f[k == code]
                pts, w = [], []
                for u, v in ((8, 12), (16, 20)):
                    (xu, wu), (xv, wv) = (qd.gauss01(int(code) >> s & 15) for s in (u, v))
                    pts.append(np.stack([np.tile(xu, len(xv)), np.repeat(xv, len(xu))], axis=1))
                    w.append(np.repeat(wv, len(wu)) * np.tile(wu, len(wv)))
                xd = disc.eval_on_elements(np.array([e]), pts[0][None])
                xd = {n: np.broadcast_to(a, (len(fs),) + a.shape[1:]) for n, a in xd.items()}
                yd = disc.eval_on_elements(fs, np.broadcast_to(pts[1], (len(fs),) + pts[1].shape))
                blk = G._blocks_tensor(xd, yd, w[0], w[1], kappa, ops)
                a = (c1 * blk["V"] + c0 * blk["Kstar"] if bc == "soft" else c0 * blk["K"] + c1 * blk["W"]) * disc.h ** 4
                for t in np.nonzero(fold[disc.el_dofs[e]] == row)[0]:
                    np.add.at(want, fold[disc.el_dofs[fs]].ravel(), a[:, t, :].ravel())
        got = np.zeros(op.n, dtype=np.complex128)
        got[col[rp[row]:rp[row + 1]]] = val[rp[row]:rp[row + 1]]
        checked += int(known.sum())
        # the same rules: the order of sums over up to 100 x 100 points and a few roundings
        # per kernel value (positions to 1e-16 of 3, regular elements no closer than
        # their size, about 0.03): 1e-12 of the largest entry
        assert np.abs(got - want)[known].max() <= 1e-12 * np.abs(got).max()
    assert checked > op.n // 2

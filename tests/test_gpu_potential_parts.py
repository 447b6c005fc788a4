"""H^2 potential: boxes of 1 to 128 points (one to many lanes per point, one or two
rounds) and sources in parts, against the direct sum."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2306_11324_amd import inputs as I


@pytest.mark.parametrize("bc", ["soft", "hard"])
@pytest.mark.parametrize("sizes", [[1], [2, 3, 5], [64, 1], [65, 43], [106, 22], [107, 128, 20], [128] * 30,
                                   [129, 300, 7]])
def test_boxes_of_every_fill(bc, sizes):
    # clusters of points around separate centres: boxes that hold a cluster or, past 128
    # points, a part of one.  q = 8 at kappa = 1: the interpolation's error (7e-9 at q = 6,
    # kappa = 8 on finer elements) and the two quadratures' difference at distances of an
    # element or more are far below 1e-6 of the largest value
    import torch
    from paper_2306_11324_amd import binding as B
    ctx = B.Context(0)
    op = B.Operator(ctx, B.Geometry(ctx, I.sphere_patches(), 3, 2), kappa=1.0, q=8,
                    bc=B.SOFT if bc == "soft" else B.HARD)
    c = torch.from_numpy(I.random_complex(7, (3, op.n))).cuda()
    rng = np.random.default_rng(len(sizes))
    centres = I.random_directions(5, len(sizes)) * 2.5
    pts = np.concatenate([x + 0.05 * rng.standard_normal((n, 3)) for x, n in zip(centres, sizes)])

    def field(what, cols):
        u = torch.full((cols.shape[0], len(pts)), float("nan"), dtype=torch.complex128, device="cuda")
        getattr(op, what)(cols, pts, u, ndir=cols.shape[0])
        torch.cuda.synchronize()
        return u.cpu().numpy()

    u = field("potential_h2", c)
    want = field("potential", c)
    assert np.abs(u - want).max() <= 1e-6 * np.abs(want).max()
    assert np.array_equal(field("potential_h2", c[1:2].contiguous())[0], u[1])

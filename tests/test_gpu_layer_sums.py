"""Far field and direct potential at the edges of their target and column blocks.

Targets are taken 64 to a wave over segments of the surface points (fewer than
24: one workgroup each), columns 1, 4 or 16 at a time; a column's values must
not depend on the other columns, and both forms must agree.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2306_11324_amd import inputs as I


@pytest.fixture(scope="module", params=["soft", "hard"])
def op(request):
    from paper_2306_11324_amd import binding as B
    ctx = B.Context(0)
    geo = B.Geometry(ctx, I.star_patches(0, 1), 3, 2)
    return B.Operator(ctx, geo, kappa=3.0, bc=B.SOFT if request.param == "soft" else B.HARD, q=4)


def evaluate(op, what, c, targets):
    import torch
    u = torch.full((c.shape[0], len(targets)), float("nan"), dtype=torch.complex128, device="cuda")
    getattr(op, what)(c, targets, u, ndir=c.shape[0])
    torch.cuda.synchronize()
    return u.cpu().numpy()


@pytest.mark.parametrize("what", ["farfield", "potential"])
@pytest.mark.parametrize("ntgt,ncol", [(1, 1), (23, 2), (24, 1), (63, 4), (64, 5), (65, 16), (257, 17), (1000, 3)])
def test_blocks_of_targets_and_columns(op, what, ntgt, ncol):
    import torch
    c = torch.from_numpy(I.random_complex(7, (ncol, op.n))).cuda()
    t = I.random_directions(11, ntgt) * (1.0 if what == "farfield" else 2.5)
    u = evaluate(op, what, c, t)
    assert np.isfinite(u).all()
    # each column alone: the same segments, the same order of sums
    one = evaluate(op, what, c[ncol - 1:].contiguous(), t)
    assert np.array_equal(u[ncol - 1], one[0])
    # the same targets one by one (workgroup form): another order of the sums over
    # 384 elements x 36 or 64 points, 1e-12 of the largest value
    k = min(ntgt, 5)
    few = evaluate(op, what, c, t[:k])
    assert np.abs(few - u[:, :k]).max() <= 1e-12 * np.abs(u).max()

"""Far field and direct potential at the edges of their target and column blocks.

Targets are taken 64 to a wave over segments of the surface points (or, for little
work, one workgroup each), columns 1, 4 or 16 at a time; a column's values must
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


@pytest.mark.parametrize("what", ["farfield", "potential"])
@pytest.mark.parametrize("m,ntgt", [(1, 1), (1, 200), (2, 64), (2, 500), (4, 3), (4, 200)])
def test_few_targets_or_points_in_either_form(what, m, ntgt):
    # a column's sums do not depend on the columns beside it on either side of the
    # rule between the forms, and a subset of targets (which may take the other form)
    # agrees to 1e-12 of the largest value
    import torch
    from paper_2306_11324_amd import binding as B
    ctx = B.Context(0)
    op = B.Operator(ctx, B.Geometry(ctx, I.sphere_patches(), m, 2), kappa=2.0, q=4, leaf_depth=1)
    c = torch.from_numpy(I.random_complex(7, (6, op.n))).cuda()
    t = I.random_directions(11, ntgt) * (1.0 if what == "farfield" else 2.5)
    u = evaluate(op, what, c, t)
    assert np.isfinite(u).all()
    for k in (0, 5):
        assert np.array_equal(evaluate(op, what, c[k:k + 1].contiguous(), t)[0], u[k])
    few = evaluate(op, what, c, t[-1:])
    assert np.abs(few - u[:, -1:]).max() <= 1e-12 * np.abs(u).max()

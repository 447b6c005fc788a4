"""fp64 blocks on either side of the rule for near field and coupling in one launch, where
nearly all products are the near field's: the same columns bit for bit, and equal to
single columns to rounding."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2306_11324_amd import inputs as I


@pytest.mark.parametrize("surface,m,leaf_depth", [("torus", 3, 2), ("torus", 2, 1), ("sphere", 4, 2)])
def test_columns_on_both_sides(surface, m, leaf_depth):
    import torch
    from paper_2306_11324_amd import binding as B
    ctx = B.Context(0)
    geo = B.Geometry(ctx, I.torus_patches() if surface == "torus" else I.sphere_patches(), m, 2)
    op = B.Operator(ctx, geo, kappa=2.0, q=4, leaf_depth=leaf_depth)
    assert op.info.far_pairs > 0
    # (level-3 torus: 100 row tiles, near share 0.98 -- one launch up to 80 columns, two beyond)
    x = torch.from_numpy(I.random_complex(7, (144, op.n))).cuda()

    def product(n):
        y = torch.full((n, op.n), float("nan"), dtype=torch.complex128, device="cuda")
        op.h2_matvec(x[:n].contiguous(), y, nrhs=n)
        torch.cuda.synchronize()
        return y.cpu().numpy()

    want = product(144)
    for n in (16, 31, 32, 64, 80, 81, 128):
        assert np.array_equal(product(n), want[:n]), n
    one = product(1)[0]
    assert np.abs(want[0] - one).max() <= 1e-12 * np.abs(one).max()

"""Near product of 2 to 15 columns on operators whose row groups hold few rows (leaf depths
0 and 1, p = 1 and 3), on either side of the rule between row groups and single rows:
bitwise the columns alone."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2306_11324_amd import inputs as I


@pytest.mark.parametrize("bc,surface,m,p,leaf_depth", [
    ("soft", "sphere", 4, 1, 0),   # 1,734 groups of a row each
    ("hard", "sphere", 4, 1, 1),
    ("soft", "sphere", 4, 3, 1),   # 1.5 rows
    ("soft", "sphere", 4, 2, 1),   # 4 rows: groups at 5 columns, rows at 7
    ("hard", "torus", 2, 2, 1),    # 250 workgroups
    ("soft", "torus", 3, 3, 2)])
def test_columns_alone(bc, surface, m, p, leaf_depth):
    import torch
    from paper_2306_11324_amd import binding as B
    ctx = B.Context(0)
    geo = B.Geometry(ctx, I.torus_patches() if surface == "torus" else I.sphere_patches(), m, p)
    op = B.Operator(ctx, geo, kappa=2.0, q=2, leaf_depth=leaf_depth, bc=B.SOFT if bc == "soft" else B.HARD)
    x = torch.from_numpy(I.random_complex(3, (15, op.n))).cuda()

    def product(cols, parts):
        y = torch.full_like(cols, float("nan"))
        op.h2_matvec(cols, y, nrhs=cols.shape[0], parts=parts)
        torch.cuda.synchronize()
        return y.cpu().numpy()

    for parts in (B.PART_NEAR, B.PART_ALL):
        one = np.concatenate([product(x[c:c + 1].contiguous(), parts) for c in range(15)])
        for n in range(2, 16):
            assert np.array_equal(product(x[:n].contiguous(), parts), one[:n]), n

"""Near product of 2 to 15 columns by row groups: every width of a pass and of a last
pass, bitwise the columns alone, and the values of the CSR."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2306_11324_amd import inputs as I


@pytest.mark.parametrize("bc,m,leaf_depth", [("soft", 4, 1), ("hard", 4, 2), ("soft", 5, 3), ("soft", 3, 1)])
def test_columns_alone_and_csr(bc, m, leaf_depth):
    import torch
    from paper_2306_11324_amd import binding as B
    ctx = B.Context(0)
    op = B.Operator(ctx, B.Geometry(ctx, I.sphere_patches(), m, 2), kappa=2.0, q=4, leaf_depth=leaf_depth,
                    bc=B.SOFT if bc == "soft" else B.HARD)
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
        if parts == B.PART_NEAR:
            near = one
    ptr, col, val = op.near_csr()
    rows = np.linspace(0, op.n - 1, 7).astype(int)
    xs = x.cpu().numpy()
    for r in rows:
        v, c = val[ptr[r]:ptr[r + 1]], col[ptr[r]:ptr[r + 1]]
        # a sum of k products: k 2^-53 of the sum of their sizes, in either order (times
        # 4 for the complex products)
        bound = 4 * len(v) * 2.0 ** -53 * (np.abs(xs[:, c]) @ np.abs(v))
        assert (np.abs(xs[:, c] @ v - near[:, r]) <= bound).all()

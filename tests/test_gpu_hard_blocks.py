"""Sound-hard fp64 products of 1 to 15 columns (stored tiles): blocks of 4, 2 and 1
columns, node groups that fill a workgroup at every degree."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2306_11324_amd import inputs as I


@pytest.mark.parametrize("q", [1, 2, 4, 7, 8, 10])
def test_columns_alone_in_blocks_and_on_the_matrix_cores(q):
    import torch
    from paper_2306_11324_amd import binding as B
    ctx = B.Context(0)
    geo = B.Geometry(ctx, I.sphere_patches(), 3, 2)
    op = B.Operator(ctx, geo, kappa=2.0, bc=B.HARD, q=q, leaf_depth=0)
    assert op.info.far_pairs > 0
    x = torch.from_numpy(I.random_complex(3, (16, op.n))).cuda()

    def product(n):
        y = torch.full((n, op.n), float("nan"), dtype=torch.complex128, device="cuda")
        op.h2_matvec(x[:n].contiguous(), y, nrhs=n, parts=B.PART_FAR)
        torch.cuda.synchronize()
        return y.cpu().numpy()

    one = np.concatenate([product(1)] + [
        op.h2_matvec(x[c:c + 1].contiguous(), torch.empty_like(x[:1]), parts=B.PART_FAR).cpu().numpy()
        for c in range(1, 15)])
    for n in (2, 3, 4, 5, 6, 7, 11, 15):
        assert np.array_equal(product(n), one[:n]), n
    # 16 columns run on the matrix cores, with the node factors outside the tiles'
    # sums: rounding apart (1e-12 of the column's largest entry, as for the blocks)
    y16 = product(16)[:15]
    assert (np.abs(y16 - one).max(axis=1) <= 1e-12 * np.abs(one).max(axis=1)).all()

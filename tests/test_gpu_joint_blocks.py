"""fp64 blocks of 16 and more columns: near field and coupling in one launch (or two),
for every column grouping and for the parts alone."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2306_11324_amd import inputs as I


@pytest.mark.parametrize("q,leaf_depth", [(2, 0), (3, 1), (6, 2), (7, 1), (10, 2)])
@pytest.mark.parametrize("ncol", [16, 33, 64])
def test_parts_and_groupings(q, leaf_depth, ncol):
    import torch
    from paper_2306_11324_amd import binding as B
    ctx = B.Context(0)
    geo = B.Geometry(ctx, I.sphere_patches(), 4, 2)
    op = B.Operator(ctx, geo, kappa=2.0, q=q, leaf_depth=leaf_depth)
    assert op.info.far_pairs > 0
    x = torch.from_numpy(I.random_complex(7, (ncol, op.n))).cuda()

    def product(parts=B.PART_ALL, shape=(0, 0), n=ncol):
        op.set_tile_shape(*shape)
        y = torch.full((n, op.n), float("nan"), dtype=torch.complex128, device="cuda")
        op.h2_matvec(x[:n].contiguous(), y, nrhs=n, parts=parts)
        torch.cuda.synchronize()
        return y.cpu().numpy()

    both = product()
    # a block's columns do not depend on its size, nor on the grouping
    assert np.array_equal(product(n=16), both[:16])
    nt = (ncol + 15) // 16
    for shape in [(c, n) for c in (1, 2, 4) for n in (1, 2, 4) if nt % c == 0 and nt % n == 0]:
        assert np.array_equal(product(shape=shape), both), shape
    # near + far: one addition per value (and the few of the far parts) apart
    near, far = product(B.PART_NEAR), product(B.PART_FAR)
    scale = np.abs(near).max(axis=1) + np.abs(far).max(axis=1)
    assert (np.abs(near + far - both).max(axis=1) <= 16 * 2.0 ** -53 * scale).all()
    # the columns one by one run on the vector path: another order of the sums
    one = np.concatenate([op.h2_matvec(x[c:c + 1].contiguous(), torch.empty_like(x[:1])).cpu().numpy()
                          for c in range(0, ncol, 5)])
    assert (np.abs(both[::5] - one).max(axis=1) <= 1e-12 * np.abs(one).max(axis=1)).all()

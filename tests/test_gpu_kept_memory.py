"""Device memory of released operators, kept for the next one of the same sizes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2306_11324_amd import inputs as I


def _product(B, torch, ctx, geo, kappa, **kw):
    op = B.Operator(ctx, geo, kappa=kappa, q=6, **kw)
    x = torch.from_numpy(I.random_complex(5, (20, op.n))).cuda()
    y = torch.empty_like(x)
    op.h2_matvec(x, y, nrhs=20)
    torch.cuda.synchronize()
    return y.cpu().numpy()


@pytest.mark.parametrize("precision", ["FP64", "MIX_BF16"])
def test_operators_in_kept_memory_are_those_in_new_memory(precision):
    import torch
    from paper_2306_11324_amd import binding as B
    kw = dict(bc=B.HARD, precision=getattr(B, precision))
    patches = I.sphere_patches()
    torch.zeros(1, device="cuda")
    new = []
    for kappa in (2.0, 3.0, 5.0):
        ctx = B.Context(0, hbm_budget=64 << 30)   # a budget: nothing is kept
        new.append(_product(B, torch, ctx, B.Geometry(ctx, patches, 5, 2), kappa, **kw))
    ctx = B.Context(0)
    geo = B.Geometry(ctx, patches, 5, 2)
    for kappa, want in zip((2.0, 3.0, 5.0), new):
        used = ctx.used_bytes()
        assert np.array_equal(_product(B, torch, ctx, geo, kappa, **kw), want), kappa
        assert ctx.used_bytes() == used


GIVEN_BACK = """
import gc
import torch
from paper_2306_11324_amd import binding as B
from paper_2306_11324_amd import inputs as I
free = []
for _ in range(3):
    ctx, other = B.Context(0), B.Context(0)
    geo = B.Geometry(ctx, I.sphere_patches(), 5, 2)
    op = B.Operator(ctx, geo, kappa=2.0, q=6)
    held = op.held_bytes()
    del op
    gc.collect()
    before = torch.cuda.mem_get_info()[0]
    del geo, ctx, other
    gc.collect()
    free.append(torch.cuda.mem_get_info()[0])
    assert held > 1 << 30 and free[-1] - before >= held // 2, (held, before, free)
assert max(free) - min(free) <= 64 << 20, free   # (streams and modules of later contexts)
"""


def test_kept_memory_is_given_back_with_the_last_context():
    # in a process of its own: contexts of other tests may be alive in this one
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", GIVEN_BACK], cwd=root, capture_output=True, text=True, timeout=90)
    assert r.returncode == 0, r.stderr

"""Device memory that the library keeps of released operators: reported, and given back
to the device for other allocators when asked."""
import gc

import pytest

pytestmark = pytest.mark.gpu

from paper_2306_11324_amd import inputs as I


def test_kept_memory_is_reported_and_given_back():
    import torch
    from paper_2306_11324_amd import binding as B
    gc.collect()
    ctx = B.Context(0)
    ctx.trim()
    assert ctx.kept_bytes() == 0
    geo = B.Geometry(ctx, I.sphere_patches(), 5, 2)
    op = B.Operator(ctx, geo, kappa=2.0, q=6)
    held = op.held_bytes()
    assert held > 1 << 30
    del op
    gc.collect()
    torch.cuda.synchronize()
    kept = ctx.kept_bytes()
    total = torch.cuda.mem_get_info()[1]
    assert held // 2 <= kept <= total // 8
    # what is kept belongs to the device, not to the context's handles
    assert ctx.used_bytes() < held and B.Context(0).kept_bytes() == kept
    free = torch.cuda.mem_get_info()[0]
    ctx.trim()
    assert ctx.kept_bytes() == 0
    # (the driver's free memory moves with its page tables too: 8 bytes per 4 KiB page)
    assert torch.cuda.mem_get_info()[0] - free >= kept - kept // 256
    # blocks come and go after it as before
    B.Operator(ctx, geo, kappa=3.0, q=6)
    gc.collect()
    assert ctx.kept_bytes() == kept
    ctx.trim()


def test_contexts_with_a_budget_keep_nothing():
    from paper_2306_11324_amd import binding as B
    gc.collect()
    ctx = B.Context(0, hbm_budget=64 << 30)
    ctx.trim()
    geo = B.Geometry(ctx, I.sphere_patches(), 5, 2)
    assert B.Operator(ctx, geo, kappa=2.0, q=6).held_bytes() > 1 << 30
    gc.collect()
    assert ctx.kept_bytes() == 0

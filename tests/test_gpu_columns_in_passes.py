"""Far field and potentials where memory is short: a block's columns go in passes, as
many at a time as there is room for partial sums of, and keep their values bit for
bit; only where one column has no room does another order of the sums stand in."""
import gc

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2306_11324_amd import inputs as I

NCOL, NTGT = 8, {"farfield": 3000, "potential": 2000, "potential_h2": 3000}
ARGS = dict(kappa=2.0, q=3, leaf_depth=1)
BUDGET = 1 << 30


class Room:
    """A context whose budget leaves a chosen number of bytes beside a level-4 operator:
    the rest is taken by the right-hand sides of a small one (13,848 bytes a direction)."""

    def __init__(self, leave):
        import torch
        from paper_2306_11324_amd import binding as B
        self.ctx = B.Context(0, hbm_budget=BUDGET)
        patches = I.sphere_patches()
        self.op = B.Operator(self.ctx, B.Geometry(self.ctx, patches, 4, 2), **ARGS)
        self.filler = B.Operator(self.ctx, B.Geometry(self.ctx, patches, 2, 2), **ARGS)
        each = self.filler.info.nelem * 9 * 16 + 3 * 8
        n = (BUDGET - self.ctx.used_bytes() - 4352 - leave) // each   # (4,352: the Gauss table)
        assert 1 <= n < 65536, n
        b = torch.empty((n, self.filler.n), dtype=torch.complex128, device="cuda")
        self.filler.cfie_rhs(np.tile([[1.0, 0.0, 0.0]], (n, 1)), b)
        torch.cuda.synchronize()
        assert leave <= BUDGET - self.ctx.used_bytes() < leave + each


def field(op, what, c, t):
    import torch
    u = torch.full((c.shape[0], len(t)), float("nan"), dtype=torch.complex128, device="cuda")
    getattr(op, what)(c, t, u, ndir=c.shape[0])
    torch.cuda.synchronize()
    return u.cpu().numpy()


def smallest(test, lo, hi, step):
    """The smallest leave in [lo, hi] (to within step) for which test(leave)."""
    assert test(hi)
    while hi - lo > step:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if test(mid) else (mid, hi)
    return hi


@pytest.mark.parametrize("what", ["farfield", "potential", "potential_h2"])
def test_room_for_one_column_is_enough(what):
    import torch
    from paper_2306_11324_amd import binding as B
    ctx = B.Context(0)
    op = B.Operator(ctx, B.Geometry(ctx, I.sphere_patches(), 4, 2), **ARGS)
    c = torch.from_numpy(I.random_complex(7, (NCOL, op.n))).cuda()
    t = I.random_directions(11, NTGT[what]) * (1.0 if what == "farfield" else 2.5)
    want = field(op, what, c, t)

    def values(leave, n):
        r = Room(leave)
        used = r.ctx.used_bytes()
        try:
            u = field(r.op, what, c[:n].contiguous(), t)
        except B.IgbError:
            return None
        finally:
            gc.collect()
        # another order of the sums at most, whatever the room
        assert np.abs(u - want[:n]).max() <= 1e-12 * np.abs(want).max()
        if what != "farfield":
            assert r.ctx.used_bytes() == used
        return u

    room = {}
    for n in (1, NCOL):
        top = 64 << 20
        accepted = smallest(lambda leave: values(leave, n) is not None, 0, top, 1 << 14)

        def same(leave):
            u = values(leave, n)
            return u is not None and np.array_equal(u, want[:n])

        room[n] = smallest(same, accepted - (1 << 14), top, 1 << 14) - accepted
    # the room beside the call's other buffers: one column's partial sums, not eight
    # columns' (two bisections to 16 KiB each, the fillers' grain)
    assert room[1] > 1 << 16
    assert abs(room[NCOL] - room[1]) <= 1 << 17


def test_far_field_leaves_no_message_and_holds_its_quadrature_only():
    import torch
    from paper_2306_11324_amd import binding as B
    r = Room(32 << 20)
    c = torch.from_numpy(I.random_complex(7, (NCOL, r.op.n))).cuda()
    t = I.random_directions(11, NTGT["farfield"])
    with pytest.raises(B.IgbError):
        r.op.farfield(c, np.zeros((1, 3)), torch.empty((NCOL, 1), dtype=torch.complex128, device="cuda"), ndir=NCOL)
    message = B._lib.igb_last_error()
    used = r.ctx.used_bytes()
    field(r.op, "farfield", c, t)
    # directions, the points' geometry (8 doubles) and densities, and the Gauss table
    points = r.op.info.nelem * 36
    held = t.size * 8 + points * 64 + NCOL * points * 16 + 4352
    assert r.ctx.used_bytes() - used == held
    assert B._lib.igb_last_error() == message


def test_a_call_that_does_without_memory_leaves_no_message():
    import torch
    from paper_2306_11324_amd import binding as B
    c, t, r = None, I.random_directions(11, NTGT["potential"]) * 2.5, None
    for leave in range(16 << 20, 32 << 20, 1 << 18):
        r = Room(leave)
        c = torch.from_numpy(I.random_complex(7, (NCOL, r.op.n))).cuda()
        u = torch.empty((NCOL, 1), dtype=torch.complex128, device="cuda")
        with pytest.raises(B.IgbError):
            r.op.potential(c, np.full((1, 3), np.nan), u, ndir=NCOL)
        message = B._lib.igb_last_error()
        try:
            field(r.op, "potential", c, t)
        except B.IgbError:
            continue
        break   # accepted with no more than 256 KiB beside its buffers
    assert B._lib.igb_last_error() == message

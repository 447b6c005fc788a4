"""Batches of the regular near-field kernel (CPU): no rule that the classification
gives runs past the rows a batch has, and the surface of the GPU test
(tests/test_gpu_near_batches.py) has the rules whose 1-D basis rows, not whose
points, bound the batch."""
import os
import shutil
import subprocess
from collections import Counter

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def bar():
    """Six bilinear patches of a 3 x 0.5 x 0.2 bar: at quad_extra = -2 elements of few
    points meet elements of many."""
    from paper_2306_11324_amd import inputs as I
    kn = np.array([0.0, 0.0, 1.0, 1.0])
    out = []
    for n, e1, e2 in I.CUBE_FACES:
        n, e1, e2 = (np.array(a, dtype=np.float64) for a in (n, e1, e2))
        net = np.ones((2, 2, 4))
        for j in range(2):
            for i in range(2):
                net[j, i, :3] = (n + (2 * i - 1) * e1 + (2 * j - 1) * e2) * (1.5, 0.25, 0.1)
        out.append(I.Patch(1, 1, kn.copy(), kn.copy(), net))
    return out


def full_batches(ptr, kind):
    """Target elements with more pairs of a (2 x 4 or 4 x 2)-point source rule, beside a
    test rule of more than 36 points, than 64 basis rows hold (10)."""
    out = []
    for e in range(len(ptr) - 1):
        k = kind[ptr[e]:ptr[e + 1]]
        for code, count in Counter((k[(k & 15) == 0] >> 8).tolist()).items():
            xu, xv, yu, yv = (code >> s & 15 for s in (0, 4, 8, 12))
            if xu * xv > 36 and sorted((yu, yv)) == [2, 4] and count > 10:
                out.append(e)
                break
    return out


def test_every_rule_fits_its_batch(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path / "near_batches")
    subprocess.run([cxx, "-std=c++17", "-I", os.path.join(ROOT, "paper_2306_11324_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "near_batches.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, check=True)
    assert r.stdout.split("\n")[:-1] == ["walked"], r.stdout


def test_the_bar_has_the_full_batches():
    from paper_2306_11324_amd import binding as B
    ctx = B.Context(B.IGB_HOST_ONLY)
    op = B.Operator(ctx, B.Geometry(ctx, bar(), 3, 1), kappa=1.0, bc=B.SOFT, q=2, eta_adm=1e6, leaf_depth=1,
                    quad_extra=-2)
    ptr, _, kind = op.near_pairs()
    assert len(full_batches(ptr, kind)) == 32

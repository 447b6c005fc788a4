"""Kept device memory on host-only contexts: there is none."""
import ctypes as C

from paper_2306_11324_amd import binding as B


def test_host_only_contexts_keep_nothing():
    ctx = B.Context(B.IGB_HOST_ONLY)
    assert ctx.kept_bytes() == 0
    ctx.trim()
    assert ctx.kept_bytes() == 0


def test_null_context():
    assert B._lib.igb_ctx_kept_bytes(C.c_void_p()) == 0
    assert B._lib.igb_ctx_trim(C.c_void_p()) == -1

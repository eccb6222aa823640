"""Calls whose usual route does not fit the caller's allocator take the one
that needs less: the build without the updates' FP16 copy.  Results as with all the
memory."""
import ctypes

import numpy as np
import pytest

from test_gpu_ham_memory import MB, _Budget

pytestmark = pytest.mark.gpu


class _Meter(_Budget):
    """Gives everything, and notes the most held at a time."""

    def __init__(self):
        super().__init__(1 << 60)
        self.peak = 0

    def _alloc(self, nbytes, ctx):
        p = super()._alloc(nbytes, ctx)
        self.peak = max(self.peak, self.used)
        return p


def _with(alloc, call):
    import paper_2510_14147_amd as fnn
    L = fnn.lib()
    L.fnn_set_allocator(alloc.a, alloc.f, None)
    try:
        return call(L)
    finally:
        L.fnn_set_allocator(fnn._alloc_cb, fnn._free_cb, None)


def test_build():
    import torch
    import paper_2510_14147_amd as fnn
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    n, d = 1_050_000, 100                    # a copy of 277 MB
    x = torch.randn(60, d, generator=gen, device="cuda").repeat(n // 60, 1)
    x += 0.1 * torch.randn(n, d, generator=gen, device="cuda")
    want = fnn.fnn_tree_export(fnn.fnn_tree_build(x, "l2"))
    fnn._bind_stream()

    def build(L):
        h = ctypes.c_void_p()
        rc = L.fnn_tree_build(ctypes.c_void_p(x.data_ptr()), n, d, 0, ctypes.byref(h))
        out = None
        if rc == 0:
            out = fnn.fnn_tree_export(fnn.Tree(h, n, d, "l2"))
        return rc, out

    m = _Meter()
    assert _with(m, build)[0] == 0 and not m.live
    b = _Budget(m.peak - 64 * MB)
    rc, got = _with(b, build)
    assert rc == 0 and b.refused > 0 and not b.live
    for k in want:
        assert np.array_equal(want[k], got[k]), k

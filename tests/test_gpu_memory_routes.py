"""Calls whose usual route does not fit the caller's allocator take the one
that needs less: the build without the updates' FP16 copy, plain tiles without
the screen's survivor list, foreign queries under a budget at every size
between.  Results as with all the memory."""
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


def _graph(L, tree, eps, o):
    import paper_2510_14147_amd as fnn
    out = ctypes.POINTER(fnn.fnn_csr)()
    return L.fnn_eps_graph_ex(tree.handle, eps, ctypes.byref(o), ctypes.byref(out)), out


def _same(alloc, out, g):
    import torch
    c = out.contents
    assert c.n == g.n and c.nnz == g.nnz
    assert torch.equal(alloc.live[c.row_ptr][:8 * (g.n + 1)].view(torch.int64), g.row_ptr)
    assert torch.equal(alloc.live[c.col][:4 * g.nnz].view(torch.int32), g.col)
    assert torch.equal(alloc.live[c.dist][:4 * g.nnz].view(torch.float32), g.dist)


def test_screened_tiles():
    import torch
    import paper_2510_14147_amd as fnn
    gen = torch.Generator(device="cuda")
    gen.manual_seed(2)
    n, d = 100_000, 20                       # little to prune: 5e9 pairs of tiles
    x = torch.randn(n, d, generator=gen, device="cuda")
    tree = fnn.fnn_tree_build(x, "l2")
    g = fnn.fnn_eps_graph(tree, 2.0, precision="fp32")
    assert g.stats["filter_pairs"] > 4e9 and g.nnz > 0
    o = fnn._options(precision="fp32")

    def query(L):
        rc, out = _graph(L, tree, 2.0, o)
        if rc == 0:
            _same(a, out, g)
            L.fnn_free(ctypes.cast(out, ctypes.c_void_p))
        return rc

    a = _Meter()
    assert _with(a, query) == 0 and not a.live
    a = _Budget(a.peak - 64 * MB)
    assert _with(a, query) == 0 and a.refused > 0 and not a.live


def test_query():
    import torch
    import paper_2510_14147_amd as fnn
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    c = 4 * torch.randn(50, 24, generator=gen, device="cuda")
    x = c.repeat(2200, 1) + 0.3 * torch.randn(110_000, 24, generator=gen, device="cuda")
    tree, q = fnn.fnn_tree_build(x[:100_000], "l2"), x[100_000:].contiguous()
    g = fnn.fnn_eps_query(tree, q, 1.6, precision="auto")
    assert g.stats["filter_pairs"] == 10 ** 9 and g.nnz > 0
    o = fnn._options(precision="auto")

    def query(L):
        out = ctypes.POINTER(fnn.fnn_csr)()
        rc = L.fnn_eps_query(tree.handle, ctypes.c_void_p(q.data_ptr()), len(q), 1.6,
                             ctypes.byref(o), ctypes.byref(out))
        if rc == 0:
            _same(a, out, g)
            L.fnn_free(ctypes.cast(out, ctypes.c_void_p))
        else:
            assert not out
        return rc

    a = _Meter()
    assert _with(a, query) == 0 and not a.live
    peak, fits = a.peak, []
    for k in range(9):
        a = _Budget(peak * k // 8)
        fits.append(_with(a, query))
        assert fits[-1] in (0, fnn.FNN_ENOMEM) and not a.live
    assert fits[0] == fnn.FNN_ENOMEM and fits[-1] == 0

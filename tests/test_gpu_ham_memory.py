"""The exact filter on codes with many neighbours where the caller's allocator
gives little more than the survivor list and the result: the same graph, with
the survivors placed as they are.  One cloud, a batch, packs of equal codes
larger than a tile, and foreign queries."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

MB = 1 << 20


class _Budget:
    """Device allocator that gives at most `budget` bytes at a time."""

    def __init__(self, budget):
        import torch
        self.torch, self.budget, self.used, self.live, self.refused = torch, budget, 0, {}, 0
        A = ctypes.CFUNCTYPE(ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p)
        F = ctypes.CFUNCTYPE(None, ctypes.c_void_p, ctypes.c_void_p)
        self.a, self.f = A(self._alloc), F(self._free)

    def _alloc(self, nbytes, ctx):
        if self.used + nbytes > self.budget:
            self.refused += 1
            return None
        t = self.torch.empty(int(nbytes), dtype=self.torch.uint8, device="cuda")
        self.used += t.numel()
        self.live[t.data_ptr()] = t
        return t.data_ptr()

    def _free(self, ptr, ctx):
        self.used -= self.live.pop(ptr).numel()


def _codes(n, groups, seed):
    rng = np.random.default_rng(seed)
    c = rng.integers(0, 2**64, (groups, 2), dtype=np.uint64)
    x = c[rng.integers(0, groups, n)]
    x[:, 0] ^= np.uint64(1) << rng.integers(0, 64, n).astype(np.uint64)
    return x


def _compare(g, call, budget):
    """The graph g against the same call under a budget of device memory."""
    import torch
    import paper_2510_14147_amd as fnn
    L, b = fnn.lib(), _Budget(budget)
    L.fnn_set_allocator(b.a, b.f, None)
    try:
        out = ctypes.POINTER(fnn.fnn_csr)()
        rc = call(L, out)
        assert rc == 0, (rc, L.fnn_last_error())
        assert b.refused > 0          # the usual way did not fit
        c = out.contents
        assert c.n == g.n and c.nnz == g.nnz
        assert torch.equal(b.live[c.row_ptr][:8 * (g.n + 1)].view(torch.int64), g.row_ptr)
        assert torch.equal(b.live[c.col][:4 * g.nnz].view(torch.int32), g.col)
        assert torch.equal(b.live[c.dist][:4 * g.nnz].view(torch.float32), g.dist)
        L.fnn_free(ctypes.cast(out, ctypes.c_void_p))
    finally:
        L.fnn_set_allocator(fnn._alloc_cb, fnn._free_cb, None)
    assert not b.live


@pytest.mark.parametrize("kind", ["one", "batch", "equal"])
def test_graph(kind):
    import paper_2510_14147_amd as fnn
    print(f"[case] {kind}", flush=True)
    n = 200_000
    x = _codes(n, 200, 1)
    if kind == "equal":
        x[1000:1500] = x[0]
    if kind == "batch":
        off = np.array([0, 60_000, 60_001, n])
        tree = fnn.fnn_tree_build_batch(x, off, "hamming")
        g = fnn.fnn_eps_graph_batch(tree, [2.0] * 3, precision="i8")
    else:
        tree = fnn.fnn_tree_build(x, "hamming")
        g = fnn.fnn_eps_graph(tree, 2.0, precision="i8")
    assert g.nnz > 1e8
    o = fnn._options(precision="i8")
    # 512 list entries a point, the result, and the call's small arrays
    budget = 8 * 512 * n + 8 * g.nnz + 3 * 256 * MB

    def call(L, out):
        if kind == "batch":
            e = (ctypes.c_double * 3)(2.0, 2.0, 2.0)
            return L.fnn_eps_graph_batch(tree.handle, e, 3, ctypes.byref(o), ctypes.byref(out))
        return L.fnn_eps_graph_ex(tree.handle, 2.0, ctypes.byref(o), ctypes.byref(out))

    _compare(g, call, budget)


def test_query():
    import torch
    import paper_2510_14147_amd as fnn
    x = _codes(220_000, 200, 2)
    tree = fnn.fnn_tree_build(x[:200_000], "hamming")
    q = torch.from_numpy(x[200_000:].view(np.int64)).cuda()
    g = fnn.fnn_eps_query(tree, q, 2.0, precision="i8")
    assert g.stats["filter_pairs"] == 200_000 * 20_000 and g.nnz > 1.9e7
    o = fnn._options(precision="i8")

    def call(L, out):
        return L.fnn_eps_query(tree.handle, ctypes.c_void_p(q.data_ptr()), len(q), 2.0,
                               ctypes.byref(o), ctypes.byref(out))

    _compare(g, call, 900 * MB)

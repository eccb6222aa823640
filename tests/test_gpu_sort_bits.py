"""Rows sorted by counting: lengths at its edges (2048 entries and below sort
in registers of a wave, up to 8192 are held, longer ones read twice), columns
within one span of 262144 and of 1048576, across several, and beyond the
2097152 of 32-bit sort keys, entries placed
packed (the filter's) and unpacked (the plain tiles')."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _cliques(n, sizes, d, seed):
    """n points far apart from each other but for cliques of the given sizes
    at random positions; returns the points and the cliques' sorted ids."""
    rng = np.random.default_rng(seed)
    x = np.zeros((n, d), np.float32)
    x[:, 0] = 8.0 * (np.arange(n) % 1024)
    x[:, 1] = 8.0 * (np.arange(n) // 1024)
    ids = rng.permutation(n)
    out, lo = [], 0
    for k, m in enumerate(sizes):
        c = np.sort(ids[lo:lo + m])
        x[c] = rng.random((m, d)).astype(np.float32) * np.float32(0.05)
        x[c, 0] -= np.float32(100.0 * (k + 1))
        out.append(c)
        lo += m
    return x, out


def _check(x, sizes, ids, **kw):
    import paper_2510_14147_amd as fnn
    print(f"[case] n={len(x)} d={x.shape[1]} sizes={sizes} {kw}", flush=True)
    g = fnn.fnn_eps_graph(fnn.fnn_tree_build(x, "l2"), 2.0, **kw)
    rp, col, dist = g.to_numpy()
    deg = np.zeros(len(x), np.int64)
    for c in ids:
        deg[c] = len(c) - 1
    assert np.array_equal(np.diff(rp), deg)
    for c in ids:
        for r in c[[0, 1, len(c) // 2, -1]]:
            want = c[c != r]
            assert np.array_equal(col[rp[r]:rp[r + 1]], want)
            ref = np.sqrt(((x[want].astype(np.float64) - x[r].astype(np.float64)) ** 2).sum(1))
            assert np.all(np.abs(dist[rp[r]:rp[r + 1]] - ref) <= 1e-5 * ref)
        for r in c:
            assert (np.diff(col[rp[r]:rp[r + 1]]) > 0).all()
    return g


@pytest.mark.parametrize("n", [40000, 262144, 262200, 1048600, 2200000])
def test_spans(n):
    sizes = [2, 40, 65, 66, 100, 129, 200, 257, 300, 513, 600, 1025, 1300, 2049, 2300, 4100]
    x, ids = _cliques(n, sizes, 3, n)
    _check(x, sizes, ids)


@pytest.mark.parametrize("kw", [{}, {"precision": "fp16"}])
@pytest.mark.parametrize("size", [2049, 2050, 8193, 8194])
def test_lengths(size, kw):
    d = 16 if kw else 3
    x, ids = _cliques(12000, [size], d, size)
    g = _check(x, [size], ids, **kw)
    if kw:
        assert g.stats["fill_path"] == 2, g.stats

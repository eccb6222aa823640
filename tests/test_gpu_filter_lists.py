"""Which pairs the matrix filters screen: every one of a single cloud (the
closed-form list, sizes around packs and groups of four of them), or those of
the traversal's list, which a trace and a batch always use (narrow packs, packs
above a tile, which the plain tiles take, and with validation).  Codes of one
to four words on both sides of the early test, and the vector formats."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _codes(n, words, seed, groups=60):
    rng = np.random.default_rng(seed)
    cent = rng.integers(0, 2**64, (groups, words), dtype=np.uint64)
    flips = rng.random((n, 64 * words)) < 0.04
    mask = np.packbits(flips, axis=1, bitorder="little").view(np.uint64)
    return np.ascontiguousarray(cent[rng.integers(0, groups, n)] ^ mask)


def _vectors(n, d, seed):
    rng = np.random.default_rng(seed)
    c = 4 * rng.normal(0, 1, (60, d))
    return (c[rng.integers(0, 60, n)] + 0.3 * rng.normal(0, 1, (n, d))).astype(np.float32)


def _check(g, x, metric, eps):
    from oracle import oracle as O
    mid = {"l2": O.L2, "angular": O.ANGULAR, "hamming": O.HAMMING}[metric]
    cmp = O.compare_csr(*g.to_numpy(), *O.bruteforce(x, mid, float(eps)), rtol=1e-5)
    assert cmp["missing"] == 0 and cmp["extra"] == 0 and cmp["ok"], cmp
    assert g.stats["validate_mismatch"] == 0
    return g.stats["filter_pairs"]


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 256, 257, 4095, 4097, 8200])
@pytest.mark.parametrize("kind", ["codes", "vectors"])
def test_every_pair(n, kind):
    import paper_2510_14147_amd as fnn
    if kind == "codes":
        x, metric, eps, prec = _codes(n, 4, n), "hamming", 24, "i8"
    else:
        x, metric, eps, prec = _vectors(n, 20, n), "l2", 1.6, "fp16"
    g = fnn.fnn_eps_graph(fnn.fnn_tree_build(x, metric), eps, precision=prec)
    assert g.stats["traverse_tests"] == 0
    assert _check(g, x, metric, eps) == n * (n - 1) // 2


@pytest.mark.parametrize("validate", [False, True])
@pytest.mark.parametrize("words,eps", [(1, 3), (2, 9), (3, 12), (4, 20), (4, 40)])
def test_codes_traversed(words, eps, validate):
    import paper_2510_14147_amd as fnn
    n = 6001
    x = _codes(n, words, 10 * words + eps)
    x[2000:2150] = x[5]                       # a pack above a tile
    g = fnn.fnn_eps_graph(fnn.fnn_tree_build(x, "hamming"), eps, precision="i8", trace=True,
                          validate=validate)
    assert 0 < _check(g, x, "hamming", eps) < n * (n - 1) // 2


@pytest.mark.parametrize("validate", [False, True])
@pytest.mark.parametrize("precision", ["fp16", "bf16", "fp8"])
@pytest.mark.parametrize("metric,d,eps", [("l2", 16, 1.3), ("l2", 100, 4.0),
                                          ("angular", 24, 0.07)])
def test_vectors_traversed(metric, d, eps, precision, validate):
    import paper_2510_14147_amd as fnn
    n = 6001
    x = _vectors(n, d, d)
    x[2000:2150] = x[5]
    g = fnn.fnn_eps_graph(fnn.fnn_tree_build(x, metric), eps, precision=precision, trace=True,
                          validate=validate)
    assert 0 < _check(g, x, metric, eps) < n * (n - 1) // 2


@pytest.mark.parametrize("words", [1, 2, 3, 4])
def test_batch_of_codes(words):
    import paper_2510_14147_amd as fnn
    sizes, eps = [2500, 1, 64, 65, 1300], [4 * words, 3, 40, 37, 2 * words]
    clouds = [_codes(m, words, i, 12) for i, m in enumerate(sizes)]
    off = np.concatenate([[0], np.cumsum(sizes)])
    tree = fnn.fnn_tree_build_batch(np.concatenate(clouds), off, "hamming")
    g = fnn.fnn_eps_graph_batch(tree, eps, precision="i8")
    rp, col, dist = g.to_numpy()
    from oracle import oracle as O
    for c, e, lo in zip(clouds, eps, off):
        s = rp[lo:lo + len(c) + 1]
        ref = O.bruteforce(c, O.HAMMING, float(e))
        assert np.array_equal(s - s[0], ref[0])
        assert np.array_equal(col[s[0]:s[-1]] - lo, ref[1])
        assert np.array_equal(dist[s[0]:s[-1]], ref[2].astype(np.float32))
    assert 0 < g.stats["filter_pairs"] <= sum(m * (m - 1) // 2 for m in sizes)

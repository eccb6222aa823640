"""Bichromatic queries that screen every (point, query) pair instead of
building a query tree: query counts around a pack of 64, data counts around a
group of four packs, every filter format, with validation, list overflow and
bad rows, against brute force on the query rows."""
import numpy as np
import pytest

from paper_2510_14147_amd import datagen as G

pytestmark = pytest.mark.gpu

MID = {"l2": 0, "angular": 1, "hamming": 2}


def _reference(P, Q, metric, eps):
    from oracle import oracle as O
    n = len(P)
    rp, col, dist = O.bruteforce(np.concatenate([P, Q]), MID[metric], eps,
                                 rows=np.arange(n, n + len(Q)))
    keep = col < n
    rows = np.repeat(np.arange(len(Q)), np.diff(rp))[keep]
    cnt = np.bincount(rows, minlength=len(Q))
    return np.concatenate([[0], np.cumsum(cnt)]), col[keep], dist[keep]


def _check(P, Q, metric, eps, **kw):
    import paper_2510_14147_amd as fnn
    from oracle import oracle as O
    tree = fnn.fnn_tree_build(P, metric)
    g = fnn.fnn_eps_query(tree, Q, eps, **kw)
    cmp = O.compare_csr(*g.to_numpy(), *_reference(P, Q, metric, eps), rtol=1e-5)
    assert cmp["ok"], cmp
    assert g.stats["validate_mismatch"] == 0
    # the rectangle, not a traversal
    assert g.stats["filter_pairs"] == len(P) * len(Q), g.stats
    return tree, g


@pytest.mark.parametrize("nq", [1, 63, 64, 65, 700])
def test_manifold_query_counts(nq):
    X = G.c2_manifold(n=24000 + nq)
    _check(X[:24000], X[24000:], "l2", 3.6, precision="auto")


@pytest.mark.parametrize("n", [20224, 20225, 20479])
@pytest.mark.parametrize("precision,validate", [("bf16", False), ("fp8", False),
                                                ("fp16", True)])
def test_manifold_formats(n, precision, validate):
    X = G.c2_manifold(n=n + 130, dim=100)
    _check(X[:n], X[n:], "l2", 3.4, precision=precision, validate=validate)


def test_angular():
    rng = np.random.default_rng(3)
    X = rng.standard_normal((21000, 24)).astype(np.float32) + 0.5
    _check(X[:20500], X[20500:], "angular", 0.9, precision="fp16")


def test_hamming():
    rng = np.random.default_rng(4)
    X = rng.integers(0, 2**64, (20700, 2), dtype=np.uint64)
    X[20600:] = X[:100] ^ np.uint64(5)
    _check(X[:20500], X[20500:], "hamming", 40, precision="auto")


def test_bad_rows_and_fp32_are_as_before():
    import paper_2510_14147_amd as fnn
    X = G.c2_manifold(n=21000)
    tree, g = _check(X[:20000], X[20000:], "l2", 3.4, precision="auto")
    q = X[20000:].copy()
    f = fnn.fnn_eps_query(tree, q, 3.4, precision="fp32")
    for a, b in zip(f.to_numpy(), g.to_numpy()):
        assert np.array_equal(a, b)      # the general path, bit for bit
    q[3, 5] = np.nan
    with pytest.raises(fnn.FnnError) as e:
        fnn.fnn_eps_query(tree, q, 3.4, precision="auto")
    assert e.value.code == fnn.FNN_EINVAL
    q[3, 5] = 1e30
    with pytest.raises(fnn.FnnError) as e:
        fnn.fnn_eps_query(tree, q, 3.4, precision="auto")
    assert e.value.code == fnn.FNN_EUNSUPPORTED

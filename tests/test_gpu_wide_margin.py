"""Filter formats whose rounding margin is far wider than the radius: they
pass nearly every pair of a cluster, so the pairs that the tree rules out must
not be screened.  Tight clusters far apart, each format set by the caller, a
projection too narrow for the data, on the set itself and for foreign
queries (the traversal's list, not every pair); and the same sets at a radius
that the margin suits, where every pair is screened.  Rows against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N, D, NQ = 20000, 16, 2000


def _clusters(sd, seed=0):
    rng = np.random.default_rng(seed)
    c = rng.normal(0, 10, (20, D))
    x = c[rng.integers(0, 20, N + NQ)] + rng.normal(0, sd, (N + NQ, D))
    return x.astype(np.float32)


def _run(x, eps, query, **kw):
    import paper_2510_14147_amd as fnn
    from oracle import oracle as O
    print(f"[case] eps={eps} query={query} {kw}", flush=True)
    tree = fnn.fnn_tree_build(x[:N], "l2")
    if query:
        g = fnn.fnn_eps_query(tree, x[N:], eps, **kw)
        f = fnn.fnn_eps_query(tree, x[N:], eps, precision="fp32")
        pairs, rows, src = N * NQ, np.arange(0, NQ, 23), x
    else:
        g = fnn.fnn_eps_graph(tree, eps, **kw)
        f = fnn.fnn_eps_graph(tree, eps, precision="fp32")
        pairs, rows, src = N * (N - 1) // 2, np.arange(0, N, 211), x[:N]
    a, b = g.to_numpy(), f.to_numpy()
    for u, v in zip(a, b):
        assert np.array_equal(u.view(np.uint8), v.view(np.uint8))
    rr, rc, _ = O.bruteforce(src, O.L2, eps, rows=rows + (N if query else 0))
    for i, r in enumerate(rows):
        want = rc[rr[i]:rr[i + 1]]
        assert np.array_equal(a[1][a[0][r]:a[0][r + 1]], want[want < N])
    assert g.nnz > 0
    return g.stats["filter_pairs"] / pairs


@pytest.mark.parametrize("query", [False, True])
@pytest.mark.parametrize("precision", ["fp16", "bf16", "fp8"])
def test_wide(precision, query):
    # |x|^2 = 1600 against eps^2 = 1.6e-5
    assert _run(_clusters(1e-3), 0.004, query, precision=precision) < 1.0


@pytest.mark.parametrize("query", [False, True])
def test_narrow_projection(query):
    x = _clusters(0.3)
    x = np.concatenate([x, x[::-1], x], axis=1)   # 48 coordinates
    assert _run(x, 3.0, query, precision="fp16", proj=16) < 1.0


@pytest.mark.parametrize("query", [False, True])
@pytest.mark.parametrize("precision", ["fp16", "auto"])
def test_selective(precision, query):
    assert _run(_clusters(1.0), 3.0, query, precision=precision) == 1.0

"""Plain-precision tiles of long lists, screened by FP16 products: row widths
around each product width, packs below and above 64 points (runs of equal
points), radii that keep few and nearly all pairs (the list overflows and the
plain tiles run), tiny and huge coordinates, an offset far larger than the
spread, a batch with its own radius per cloud and a query against a kept
tree.  Rows must be the oracle's, and the same bit for bit as those of the
filters' exact decision where a filter takes the same set."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _points(n, d, seed, scale=1.0, offset=0.0):
    rng = np.random.default_rng(seed)
    k = 40
    c = rng.normal(0, 1, (k, d))
    w = 1.0 / np.arange(1, k + 1)
    lab = rng.choice(k, n, p=w / w.sum())
    x = c[lab] + rng.normal(0, 1, (n, d)) * 10.0 ** rng.uniform(-2, -0.7, k)[lab][:, None]
    x[n // 2: n // 2 + 150] = x[0]
    return (x * scale + offset).astype(np.float32)


def _radius(x, frac, seed=0):
    r = np.random.default_rng(seed).choice(len(x), 100, replace=False)
    q = ((x[r, None].astype(np.float64) - x[None, ::23]) ** 2).sum(2)
    return float(np.sqrt(np.quantile(q, frac)))


def _rows(O, g, x, mid, eps, rows, symmetric=True):
    """Rows of the graph against the oracle's."""
    rp, col, dist = g.to_numpy()
    ref = O.bruteforce(x, mid, eps, rows=rows)
    got = np.concatenate([np.arange(rp[r], rp[r + 1]) for r in rows])
    sub = np.concatenate([[0], np.cumsum(rp[rows + 1] - rp[rows])])
    cmp = O.compare_csr(sub, col[got], dist[got], *ref, rtol=1e-5)
    assert cmp["missing"] == 0 and cmp["extra"] == 0 and cmp["ok"], cmp
    assert not symmetric or O.csr_symmetric(rp, col, dist)


@pytest.mark.parametrize("d", [15, 16, 17, 32, 33, 55, 64, 65, 100, 128, 130])
def test_l2(d):
    import paper_2510_14147_amd as fnn
    from oracle import oracle as O
    print(f"[case] d={d}", flush=True)
    x = _points(30001, d, d)
    eps = _radius(x, 0.001)
    tree = fnn.fnn_tree_build(x, "l2")
    g = fnn.fnn_eps_graph(tree, eps, precision="fp32")
    screened = g.stats["filter_pairs"]
    assert (screened > 0) == (d <= 128), g.stats
    assert g.stats["precision_used"] == 0
    rows = np.sort(np.random.default_rng(d).choice(len(x), 600, replace=False))
    _rows(O, g, x, O.L2, eps, rows)
    if d <= 128:
        f = fnn.fnn_eps_graph(tree, eps, precision="fp16")
        for u, v in zip(g.to_numpy(), f.to_numpy()):
            assert np.array_equal(u.view(np.uint8), v.view(np.uint8))


@pytest.mark.parametrize("scale,offset", [(1e-7, 0.0), (1e5, 0.0), (1.0, 1000.0)])
@pytest.mark.parametrize("d,frac", [(20, 0.002), (60, 0.02), (40, 0.5), (40, 1.0)])
def test_scales_and_radii(d, frac, scale, offset):
    import paper_2510_14147_amd as fnn
    from oracle import oracle as O
    print(f"[case] d={d} frac={frac} scale={scale} offset={offset}", flush=True)
    x = _points(24000 if frac < 0.1 else 9000, d, d, scale, offset)
    eps = _radius(x, frac)
    g = fnn.fnn_eps_graph(fnn.fnn_tree_build(x, "l2"), eps, precision="fp32")
    rows = np.sort(np.random.default_rng(d).choice(len(x), 200, replace=False))
    _rows(O, g, x, O.L2, eps, rows, frac < 0.1)


@pytest.mark.parametrize("d,eps", [(16, 0.05), (50, 0.1), (128, 0.02)])
def test_angular(d, eps):
    import paper_2510_14147_amd as fnn
    from oracle import oracle as O
    print(f"[case] d={d}", flush=True)
    x = _points(30001, d, d + 5)
    g = fnn.fnn_eps_graph(fnn.fnn_tree_build(x, "angular"), eps, precision="fp32")
    rows = np.sort(np.random.default_rng(d).choice(len(x), 400, replace=False))
    _rows(O, g, x, O.ANGULAR, eps, rows)


def test_batch():
    import paper_2510_14147_amd as fnn
    from oracle import oracle as O
    sizes, d = [9000, 1, 700, 8000, 65], 24
    clouds = [_points(max(n, 400), d, n)[:n] for n in sizes]
    eps = [0.3 + 0.05 * i for i in range(len(sizes))]
    off = np.cumsum([0] + sizes).astype(np.int64)
    tree = fnn.fnn_tree_build_batch(np.concatenate(clouds), off, "l2")
    g = fnn.fnn_eps_graph_batch(tree, eps, precision="fp32")
    rp, col, dist = g.to_numpy()
    for c, e, lo in zip(clouds, eps, off):
        s = rp[lo:lo + len(c) + 1]
        ref = O.bruteforce(c, O.L2, e)
        cmp = O.compare_csr(s - s[0], col[s[0]:s[-1]] - lo, dist[s[0]:s[-1]], *ref, rtol=1e-5)
        assert cmp["missing"] == 0 and cmp["extra"] == 0 and cmp["ok"], cmp


def test_query():
    import paper_2510_14147_amd as fnn
    from oracle import oracle as O
    x = _points(44000, 24, 3)
    p, q = x[:30000], x[30000:]
    eps = _radius(x, 0.001)
    g = fnn.fnn_eps_query(fnn.fnn_tree_build(p, "l2"), q, eps, precision="fp32")
    rp, col, dist = g.to_numpy()
    assert len(rp) == len(q) + 1
    rows = np.arange(30000, 44000, 41)
    rr, rc, rd = O.bruteforce(x, O.L2, eps, rows=rows)
    for i, r in enumerate(rows - 30000):
        keep = rc[rr[i]:rr[i + 1]] < 30000
        assert np.array_equal(col[rp[r]:rp[r + 1]], rc[rr[i]:rr[i + 1]][keep])
        ref = rd[rr[i]:rr[i + 1]][keep]
        assert np.all(np.abs(dist[rp[r]:rp[r + 1]] - ref) <= 1e-5 * ref)

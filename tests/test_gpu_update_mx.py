"""Net selection where its distances are screened by FP16 products: row
widths around each product width (and just outside the screened range), hubs
below and above a chunk of 64 points and a batch of 32 centres, duplicates,
tiny and huge coordinates and an offset far larger than the spread.  Every
point must sit under the nearest of its siblings' centres, the cover tree
must satisfy its invariants and the graph must be the oracle's."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _points(n, d, seed, scale=1.0, offset=0.0):
    rng = np.random.default_rng(seed)
    k = max(2, n // 150)
    c = rng.normal(0, 1, (k, d))
    # cluster sizes from a few points to most of a level
    w = 1.0 / np.arange(1, k + 1)
    lab = rng.choice(k, n, p=w / w.sum())
    x = c[lab] + rng.normal(0, 1, (n, d)) * 10.0 ** rng.uniform(-3, -0.5, (n, 1))
    x[n // 2: n // 2 + n // 40] = x[0]
    return (x * scale + offset).astype(np.float32)


def _nearest(x, t):
    """Points not under the nearest sibling centre, to the rounding of an
    FP32 sum of d squares (each of d + 3 operations 2^-24, both sides)."""
    d = x.shape[1]
    tol = 2.0 * (d + 3) * 2.0 ** -24
    xd, bad = x.astype(np.float64), 0
    for v in range(t["nnodes"]):
        cb, m = t["child_begin"][v], t["child_count"][v]
        if m < 2:
            continue
        ch = np.arange(cb, cb + m)
        c = xd[t["center"][ch]]
        b, e = t["pt_begin"][ch], t["pt_end"][ch]
        if (e - b).sum() != t["pt_end"][v] - t["pt_begin"][v]:
            return -1
        for j, u in enumerate(ch):
            p = xd[t["order"][t["pt_begin"][u]:t["pt_end"][u]]]
            for i in range(0, len(p), 256):
                q = ((p[i:i + 256, None, :] - c[None]) ** 2).sum(2)
                bad += int((q[:, j] > q.min(1) * (1 + tol)).sum())
    return bad


def _check(fnn, O, x, metric, mid, eps, zeta, nearest, **kw):
    tree = fnn.fnn_tree_build(x, metric, zeta=zeta, **kw)
    rp, col, dist = fnn.fnn_eps_graph(tree, eps).to_numpy()
    t = fnn.fnn_tree_export(tree)
    if nearest:
        assert _nearest(x, t) == 0
    t["radius"] = t["radius"].astype(np.float64)
    v = O.check_tree(x, mid, t)
    assert all(c == 0 for c in v.values()), v
    cmp = O.compare_csr(rp, col, dist, *O.bruteforce(x, mid, eps), rtol=1e-5)
    assert cmp["missing"] == 0 and cmp["extra"] == 0 and cmp["ok"], cmp


@pytest.mark.parametrize("d", [12, 16, 17, 32, 33, 64, 65, 100, 128, 132])
@pytest.mark.parametrize("n,zeta", [(90, 8), (2500, 64)])
def test_l2(d, n, zeta):
    import paper_2510_14147_amd as fnn
    from oracle import oracle as O
    print(f"[case] d={d} n={n}", flush=True)
    x = _points(n, d, 31 * d + n)
    _check(fnn, O, x, "l2", O.L2, 0.3 * d ** 0.5, zeta, True)


@pytest.mark.parametrize("kmax", [1, 31, 33, 64, 65, 200, 256])
@pytest.mark.parametrize("n,d,metric", [(6000, 20, "l2"), (6000, 64, "angular"), (40000, 16, "l2")])
def test_candidates_per_pass(n, d, metric, kmax):
    """Conflict blocks of 32 candidates, their keys cut by a threshold first
    (more than 256 chunks) or not."""
    import paper_2510_14147_amd as fnn
    from oracle import oracle as O
    print(f"[case] n={n} d={d} {metric} kmax={kmax}", flush=True)
    x = _points(n, d, d + kmax)
    t = fnn.fnn_tree_export(fnn.fnn_tree_build(x, metric, kmax=kmax))
    t["radius"] = t["radius"].astype(np.float64)
    v = O.check_tree(x, O.L2 if metric == "l2" else O.ANGULAR, t)
    assert all(c == 0 for c in v.values()), v


@pytest.mark.parametrize("scale,offset", [(1e-7, 0.0), (1e5, 0.0), (1.0, 1000.0)])
@pytest.mark.parametrize("d", [20, 60])
def test_scales(d, scale, offset):
    import paper_2510_14147_amd as fnn
    from oracle import oracle as O
    print(f"[case] d={d} scale={scale} offset={offset}", flush=True)
    x = _points(2000, d, d, scale, offset)
    _check(fnn, O, x, "l2", O.L2, 0.3 * d ** 0.5 * scale, 16, True)


@pytest.mark.parametrize("d", [16, 50, 128])
def test_angular(d):
    import paper_2510_14147_amd as fnn
    from oracle import oracle as O
    print(f"[case] d={d}", flush=True)
    _check(fnn, O, _points(2000, d, d + 5), "angular", O.ANGULAR, 0.3, 32, False)


@pytest.mark.parametrize("d", [16, 40])
def test_batch(d):
    import paper_2510_14147_amd as fnn
    from oracle import oracle as O
    print(f"[case] d={d}", flush=True)
    sizes, eps = [700, 1, 65, 900, 64, 30], 0.3 * d ** 0.5
    clouds = [_points(max(n, 50), d, n + d)[:n] for n in sizes]
    off = np.cumsum([0] + sizes).astype(np.int64)
    tree = fnn.fnn_tree_build_batch(np.concatenate(clouds), off, "l2", zeta=16)
    rp, col, dist = fnn.fnn_eps_graph_batch(tree, [eps] * len(clouds)).to_numpy()
    lo = 0
    for c in clouds:
        s = rp[lo:lo + len(c) + 1]
        ref = O.bruteforce(c, O.L2, eps)
        cmp = O.compare_csr(s - s[0], col[s[0]:s[-1]] - lo, dist[s[0]:s[-1]], *ref, rtol=1e-5)
        assert cmp["missing"] == 0 and cmp["extra"] == 0 and cmp["ok"], cmp
        lo += len(c)


@pytest.mark.parametrize("kmax,d", [(64, 3), (200, 3), (64, 16)])
def test_sliced_candidates(kmax, d):
    """A hub of more than 16384 chunks (its candidates are cut per slice
    first): the root's children are more than half its radius bound apart and
    hold every point within that of their centres."""
    import paper_2510_14147_amd as fnn
    print(f"[case] kmax={kmax} d={d}", flush=True)
    x = np.random.default_rng(kmax + d).random((1100000, d)).astype(np.float32)
    t = fnn.fnn_tree_export(fnn.fnn_tree_build(x, "l2", kmax=kmax))
    half = 2.0 ** (int(t["level"][0]) - 1)
    ch = np.arange(t["child_begin"][0], t["child_begin"][0] + t["child_count"][0])
    assert len(ch) > 1
    c = x[t["center"][ch]].astype(np.float64)
    dist = np.sqrt(((c[:, None] - c[None]) ** 2).sum(2))
    np.fill_diagonal(dist, np.inf)
    assert dist.min() > half
    assert t["pt_begin"][ch[0]] == 0 and t["pt_end"][ch[-1]] == len(x)
    assert np.array_equal(t["pt_begin"][ch[1:]], t["pt_end"][ch[:-1]])
    assert np.array_equal(np.sort(t["order"]), np.arange(len(x)))
    far = 0.0
    for k, u in enumerate(ch):
        p = x[t["order"][t["pt_begin"][u]:t["pt_end"][u]]].astype(np.float64)
        far = max(far, float(np.sqrt(((p - c[k]) ** 2).sum(1)).max()))
    assert far <= half

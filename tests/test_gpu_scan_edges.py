"""Trees whose levels sit around the one-launch scan (8192 values) and the
tile of the general one, the passes that run before a level's graph, and the
closed-form list's run table past one wave of runs."""
import numpy as np
import pytest

from paper_2510_14147_amd import datagen as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [65, 1024, 8191, 8192, 8193, 20001])
@pytest.mark.parametrize("graph_passes", [None, 1, 2])
def test_same_tree_and_graph_at_scan_edges(n, graph_passes):
    import paper_2510_14147_amd as fnn
    from oracle import oracle as O
    x = G.random_points(n, 3, seed=n, duplicates=n // 50)
    a = fnn.fnn_tree_export(fnn.fnn_tree_build(x, "l2", zeta=2, graph_passes=8))
    t = fnn.fnn_tree_build(x, "l2", zeta=2, graph_passes=graph_passes)
    b = fnn.fnn_tree_export(t)
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    eps = 0.6 * n ** (-1 / 3)
    rows = np.arange(0, n, max(1, n // 700))
    rp, col, dist = fnn.fnn_eps_graph(t, eps).to_numpy()
    r2, c2, d2 = O.bruteforce(x, O.L2, eps, rows=rows)
    assert np.array_equal(np.diff(rp)[rows], np.diff(r2))
    assert np.array_equal(np.concatenate([col[rp[r]:rp[r + 1]] for r in rows]), c2)


def test_closed_form_list_past_one_wave_of_runs():
    # 64 runs of 64 packs of 64 rows are 262144 points
    import paper_2510_14147_amd as fnn
    x = G.c2_manifold(n=262144 + 64 * 64 + 1, dim=32)
    t = fnn.fnn_tree_build(x, "l2")
    g = fnn.fnn_eps_graph(t, 0.9, precision="fp16")
    h = fnn.fnn_eps_graph(t, 0.9, precision="fp32")
    assert g.stats["filter_pairs"] == g.n * (g.n - 1) // 2
    for u, v in zip(g.to_numpy(), h.to_numpy()):
        assert np.array_equal(u.view(np.uint8), v.view(np.uint8))

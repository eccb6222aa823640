"""Packs where runs of children cannot share one: leaf blocks above half a
pack, packs of one point, batches of many small clouds (whose roots never
share a pack), alone and between blocks that do share, against the next-fit
rule replayed on the exported tree."""
import numpy as np
import pytest

from test_gpu_packs import next_fit_packs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("zeta,pack", [(64, 1), (64, 40), (33, 64), (16, 64), (3, 5), (1, 2)])
def test_one_cloud(zeta, pack):
    import paper_2510_14147_amd as fnn
    rng = np.random.default_rng(zeta + pack)
    # groups of equal points (blocks of 1 to 60) around many centres
    k = rng.integers(1, 61, 700)
    x = np.repeat(rng.random((700, 16)).astype(np.float32), k, axis=0)
    x = x[rng.permutation(len(x))]
    tree = fnn.fnn_tree_build(x, "l2", zeta=zeta, pack=pack)
    want, maxcc = next_fit_packs(fnn.fnn_tree_export(tree), pack, -1)
    assert maxcc > 64 and tree.stats["packs"] == want


@pytest.mark.parametrize("nclouds", [63, 64, 65, 129, 4000])
def test_small_clouds(nclouds):
    import paper_2510_14147_amd as fnn
    from oracle import oracle as O
    rng = np.random.default_rng(nclouds)
    sizes = rng.integers(1, 90, nclouds)     # some above a leaf block of 64
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    x = rng.random((int(off[-1]), 3)).astype(np.float32)
    tree = fnn.fnn_tree_build_batch(x, off, "l2")
    want, _ = next_fit_packs(fnn.fnn_tree_export(tree), 64, 0)
    assert tree.stats["packs"] == want
    rp, col, dist = fnn.fnn_eps_graph_batch(tree, [0.2] * nclouds).to_numpy()
    for c in rng.choice(nclouds, 20, replace=False):
        a, b = off[c], off[c + 1]
        ref = O.bruteforce(x[a:b], O.L2, 0.2)
        s = rp[a:b + 1]
        cmp = O.compare_csr(s - s[0], col[s[0]:s[-1]] - a, dist[s[0]:s[-1]], *ref, rtol=1e-5)
        assert cmp["ok"], cmp

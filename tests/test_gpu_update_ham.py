"""Net selection over codes at the edges of its register widths (one word up
to 512 bits, and beyond), with hubs below and above a chunk and more new
centres than a wave's 64 in one pass: every point must sit under a nearest
sibling centre (the first of equals), the tree must satisfy its invariants
and the graph must be the oracle's."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("words", [1, 2, 3, 4, 5, 8, 9])
@pytest.mark.parametrize("n,kmax", [(70, 64), (3000, 64), (3000, 200)])
def test_codes(words, n, kmax):
    import paper_2510_14147_amd as fnn
    from oracle import oracle as O
    print(f"[case] words={words} n={n} kmax={kmax}", flush=True)
    rng = np.random.default_rng(words * n + kmax)
    cent = rng.integers(0, 2**64, (n // 10, words), dtype=np.uint64)
    flips = np.packbits(rng.random((n, 64 * words)) < 0.05, axis=1, bitorder="little")
    x = np.ascontiguousarray(cent[rng.integers(0, len(cent), n)] ^ flips.view(np.uint64))
    eps = 6.0 * words
    tree = fnn.fnn_tree_build(x, "hamming", zeta=8, kmax=kmax)
    rp, col, dist = fnn.fnn_eps_graph(tree, eps).to_numpy()
    ref = O.bruteforce(x, O.HAMMING, eps)
    assert np.array_equal(rp, ref[0]) and np.array_equal(col, ref[1])
    assert np.array_equal(dist, ref[2].astype(np.float32))
    t = fnn.fnn_tree_export(tree)
    bits = np.unpackbits(x.view(np.uint8), axis=1).astype(np.int32)
    for v in np.flatnonzero(t["child_count"]):
        ch = np.arange(t["child_begin"][v], t["child_begin"][v] + t["child_count"][v])
        c = bits[t["center"][ch]]
        for j, u in enumerate(ch):
            p = bits[t["order"][t["pt_begin"][u]:t["pt_end"][u]]]
            d = p @ (1 - c).T + (1 - p) @ c.T
            assert (d.argmin(1) == j).all()
    t["radius"] = t["radius"].astype(np.float64)
    assert all(k == 0 for k in O.check_tree(x, O.HAMMING, t).values())

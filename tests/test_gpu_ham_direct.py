"""The matrix-core filter for Hamming codes: one to four words, radii on both
sides of the early test's limit (36) and of half the code length, sizes
around a pack of 64 on the closed-form list (256 packs or more) and on the
traversal's, with validation and without, against brute force."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _codes(n, words, seed):
    rng = np.random.default_rng(seed)
    cent = rng.integers(0, 2**64, (max(2, n // 40), words), dtype=np.uint64)
    flips = rng.random((n, 64 * words)) < 0.06
    mask = np.packbits(flips, axis=1, bitorder="little").view(np.uint64)
    return np.ascontiguousarray(cent[rng.integers(0, len(cent), n)] ^ mask)


def _check(x, eps, **kw):
    import paper_2510_14147_amd as fnn
    from oracle import oracle as O
    tree = fnn.fnn_tree_build(x, "hamming")
    g = fnn.fnn_eps_graph(tree, eps, precision="i8", **kw)
    rp, col, dist = g.to_numpy()
    ref = O.bruteforce(x, O.HAMMING, float(eps))
    assert np.array_equal(rp, ref[0]) and np.array_equal(col, ref[1])
    assert np.array_equal(dist, ref[2].astype(np.float32))
    return g


@pytest.mark.parametrize("n", [65, 1000, 1023, 1025])
@pytest.mark.parametrize("words,eps", [(1, 3), (1, 40), (2, 12), (3, 20), (3, 38), (4, 24),
                                       (4, 36), (4, 37), (4, 100), (4, 130)])
def test_words_and_radii(n, words, eps):
    g = _check(_codes(n, words, 100 * words + eps), eps)
    if n < 1000:
        g = _check(_codes(n, words, 7 * words + eps), eps, validate=True)
        assert g.stats["validate_mismatch"] == 0


@pytest.mark.parametrize("n", [16384, 16385, 16447])
@pytest.mark.parametrize("words,eps", [(1, 6), (3, 20), (4, 24), (4, 40)])
def test_closed_form_list(n, words, eps):
    # unrelated codes: the traversal could prune little
    g = _check(_codes(n, words, n + words), eps)
    if g.stats["packs"] >= 256 and g.stats["traverse_tests"] == 8192:
        assert g.stats["filter_pairs"] == n * (n - 1) // 2


def test_duplicates_and_foreign_queries():
    import paper_2510_14147_amd as fnn
    from oracle import oracle as O
    x = _codes(3000, 4, 5)
    x[1000:1200] = x[7]          # a pack of equal codes larger than a tile
    _check(x, 24)
    q = _codes(333, 4, 6)
    q[::3] = x[:111] ^ np.uint64(1)
    tree = fnn.fnn_tree_build(x, "hamming")
    rp, col, dist = fnn.fnn_eps_query(tree, q, 24.0, precision="i8").to_numpy()
    r2, c2, d2 = O.bruteforce(np.concatenate([x, q]), O.HAMMING, 24.0,
                              rows=np.arange(3000, 3333))
    keep = c2 < 3000
    rows = np.repeat(np.arange(333), np.diff(r2))[keep]
    assert np.array_equal(np.diff(rp), np.bincount(rows, minlength=333))
    assert np.array_equal(col, c2[keep]) and np.array_equal(dist, d2[keep].astype(np.float32))

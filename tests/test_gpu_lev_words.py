"""Edit distance at the edges of its bit vectors: string lengths around the
32-bit word boundaries up to 256 symbols, alphabets around the 2, 5 and 8
bit planes, rows that are not a multiple of four bytes, empty strings, and
levels with few hubs (conflict tests of their own) and with many."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _strings(n, stride, alphabet, seed):
    rng = np.random.default_rng(seed)
    out = np.full((n, stride), 0xFF, np.uint8)
    fam = [rng.integers(0, alphabet, rng.integers(max(1, stride - 40), stride + 1))
           for _ in range(max(2, n // 12))]
    for i in range(n):
        s = list(fam[rng.integers(len(fam))])
        for _ in range(rng.integers(0, 5)):
            p = int(rng.integers(0, max(1, len(s))))
            k = rng.integers(0, 3)
            if k == 0 and s:
                s[p] = int(rng.integers(0, alphabet))
            elif k == 1:
                s.insert(p, int(rng.integers(0, alphabet)))
            elif s:
                del s[p]
        s = s[:stride]
        out[i, :len(s)] = s
    out[n // 2, :] = 0xFF  # an empty string
    return out


@pytest.mark.parametrize("stride,alphabet,eps", [
    (31, 4, 4), (32, 1, 2), (33, 5, 5), (64, 20, 6), (65, 33, 4), (96, 32, 6),
    (97, 2, 5), (130, 4, 6), (193, 254, 8), (256, 4, 7), (256, 255, 4)])
@pytest.mark.parametrize("zeta", [4, 64])
def test_matches_oracle(stride, alphabet, eps, zeta):
    import paper_2510_14147_amd as fnn
    from oracle import oracle as O
    x = _strings(900, stride, alphabet, 7 * stride + alphabet)
    tree = fnn.fnn_tree_build(x, "levenshtein", zeta=zeta)
    rp, col, dist = fnn.fnn_eps_graph(tree, eps).to_numpy()
    ref = O.bruteforce(x, O.LEVENSHTEIN, float(eps))
    assert np.array_equal(rp, ref[0]) and np.array_equal(col, ref[1])
    assert np.array_equal(dist, ref[2].astype(np.float32))

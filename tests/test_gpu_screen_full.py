"""Screened plain tiles whose survivors outgrow their list: long lists that a
sample sends to the tiles, shorter ones whose screen ends where the list
overflows, blocks that pass whole, and lists cut short by the caller, each
against the oracle on sampled rows; sparse sets beside them stay screened."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _run(n, d, sd, eps, screened, **kw):
    import paper_2510_14147_amd as fnn
    from oracle import oracle as O
    print(f"[case] n={n} d={d} sd={sd} eps={eps} {kw}", flush=True)
    rng = np.random.default_rng(n + d)
    x = (rng.normal(0, 1, (30, d))[rng.integers(0, 30, n)] +
         rng.normal(0, sd, (n, d))).astype(np.float32)
    g = fnn.fnn_eps_graph(fnn.fnn_tree_build(x, "l2"), eps, precision="fp32", **kw)
    assert (g.stats["filter_pairs"] > 0) == screened, g.stats
    rp, col, dist = g.to_numpy()
    rows = np.sort(rng.choice(n, 40, replace=False))
    got = np.concatenate([np.arange(rp[r], rp[r + 1]) for r in rows])
    sub = np.concatenate([[0], np.cumsum(rp[rows + 1] - rp[rows])])
    cmp = O.compare_csr(sub, col[got], dist[got], *O.bruteforce(x, O.L2, eps, rows=rows),
                        rtol=1e-5)
    assert cmp["missing"] == 0 and cmp["extra"] == 0 and cmp["ok"], cmp


@pytest.mark.parametrize("d", [16, 40])
@pytest.mark.parametrize("n", [9000, 40000])
def test_rates(n, d):
    u = np.sqrt(2.0 * d)
    _run(n, d, 1.0, 0.45 * u, True)           # few pairs
    _run(n, d, 1.0, 1.35 * u, False)          # about half of them
    _run(n, d, 1e-3, 6.0 * u, False)          # every one


@pytest.mark.parametrize("cap,screened", [(1, False), (1000, False), (100000, True)])
def test_list_cap(cap, screened):
    # some 5000 edges
    _run(12000, 24, 1.0, 0.6 * np.sqrt(48.0), screened, list_cap=cap)

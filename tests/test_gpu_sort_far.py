"""Long rows whose columns lie many millions apart (counted windows against
sorts in a work-group's registers): lengths at the edges of each, in a random
order of the points and in cliques of consecutive ids, placed unpacked by the
plain tiles and packed by the filter."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _check(n, d, sizes, random, noise, **kw):
    import torch
    import paper_2510_14147_amd as fnn
    print(f"[case] n={n} d={d} sizes={sizes} random={random} {kw}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    if noise:      # points far apart in every direction
        x = torch.randn(n, d, generator=gen, device="cuda") * 6
    else:          # a plane grid
        x = torch.zeros(n, d, device="cuda")
        i = torch.arange(n, device="cuda")
        x[:, 0] = 8.0 * (i % 4096).float()
        x[:, 1] = 8.0 * (i // 4096).float()
    ids = torch.randperm(n, generator=gen, device="cuda") if random else \
        torch.arange(n, device="cuda") + 0
    out, lo = [], 0 if random else n // 2 - 5000
    for k, m in enumerate(sizes):
        c = ids[lo:lo + m].sort().values
        p = torch.rand(m, d, generator=gen, device="cuda") * 0.05
        if noise:
            x[c] = x[c[0]] + p
        else:
            p[:, 0] -= 100.0 * (k + 1)
            x[c] = p
        out.append(c)
        lo += m
    g = fnn.fnn_eps_graph(fnn.fnn_tree_build(x, "l2"), 2.0, **kw)
    rp, col, dist = g.row_ptr, g.col, g.dist
    deg = torch.zeros(n, dtype=torch.int64, device="cuda")
    for c in out:
        deg[c] = len(c) - 1
    assert torch.equal(rp[1:] - rp[:-1], deg)
    for c in out:
        for r in c[np.linspace(0, len(c) - 1, 40).astype(int)].tolist():
            a, b = int(rp[r]), int(rp[r + 1])
            want = c[c != r]
            assert torch.equal(col[a:b].long(), want)
            ref = (x[want].double() - x[r].double()).norm(dim=1)
            assert bool(((dist[a:b] - ref).abs() <= 1e-5 * ref).all())
    return g


@pytest.mark.parametrize("n,random", [(5000000, True), (17900000, True), (17900000, False)])
def test_unpacked(n, random):
    _check(n, 3, [2049, 2100, 4096, 4097, 8192, 8193, 16384, 16386], random, False)


def test_packed():
    g = _check(4300000, 16, [2049, 4096, 4097, 8300], True, True, precision="fp16")
    assert g.stats["fill_path"] == 2

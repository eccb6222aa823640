"""Calls from several threads at once, each on a stream of its own, with and
without recorded launch sequences: the results of one thread."""
import threading

import pytest

pytestmark = pytest.mark.gpu


def _job(t, passes):
    import torch
    import paper_2510_14147_amd as fnn
    out, s = [], torch.cuda.Stream()
    with torch.cuda.stream(s):
        for i in range(5):
            gen = torch.Generator(device="cuda")
            gen.manual_seed(100 * t + i)
            d = (3, 16, 40, 128)[(t + i) % 4]
            c = torch.randn(40, d, generator=gen, device="cuda")
            x = c.repeat(500, 1) + 0.1 * torch.randn(20000, d, generator=gen, device="cuda")
            s.synchronize()
            tree = fnn.fnn_tree_build(x, "l2", graph_passes=passes)
            g = fnn.fnn_eps_graph(tree, 0.12 * d ** 0.5, precision=("fp32", "auto")[i % 2],
                                  graph_passes=passes)
            out.append([v.cpu().clone() for v in (g.row_ptr, g.col, g.dist)])
    return out


@pytest.mark.parametrize("passes", [None, 1, 2])
def test_threads(passes):
    import torch
    want = [_job(t, passes) for t in range(4)]
    got, errors = [None] * 4, []

    def run(t):
        try:
            got[t] = _job(t, passes)
        except Exception as e:  # reported below
            errors.append(e)

    th = [threading.Thread(target=run, args=(t,)) for t in range(4)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not errors, errors
    for a, b in zip(want, got):
        for u, v in zip(a, b):
            assert all(torch.equal(x, y) for x, y in zip(u, v))
    assert min(len(u[1]) for a in want for u in a) > 0

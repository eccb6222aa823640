"""The work that users of this library have it do, as measurable cases.

A case is a dict of plain values.  ``listed()`` gives the fixed ones, ``draw``
one more of the same ranges; ``prepare`` makes what a program holds before the
call (points on the device, the radius, a tree it keeps), ``run`` is one pass
through the public entry points, ``work`` the bytes and operations no
implementation can do without, and ``exact`` the same outputs from plain torch
in 64 bits.

``kind`` is the shape of the call:

* ``graph``     cover tree of new points, then their epsilon-graph;
* ``requery``   the epsilon-graph of a tree that the program already has
                (several radii over one set);
* ``query``     new points against a kept tree (bichromatic);
* ``batch``     many independent clouds in one forest, a radius for each;
* ``landmark``  the graph by Voronoi cells and their ghosts;
* ``model``     the cost model's inference and its full-batch gradient.

``data`` is the recipe of the points, the same as the package's generators
(``datagen.py``), drawn on the device.  Radii are calibrated on sample rows
for a target mean neighbour count, as the package's workloads are; codes and
strings take theirs as given.

A case fixes the cloud, a seed its pose: the order of the rows (and with it
the tree's root and all that follows), the order and signs of the axes, the
order and values of the bits, the names of the symbols.  Distances, and so
the length of the result, are the same for every seed; rows, columns and
trees are not.
"""
import math
import zlib

import numpy as np
import torch

import paper_2510_14147_amd as fnn

MLP_SHAPES = ((64, 16), (64,), (64, 64), (64,), (2, 64), (2,))


def listed():
    return [
        # the smallest cloud of the many-clouds workload, 3-d, by itself:
        # launches and host round trips are all of its time
        dict(name="cloud_1k_d3", kind="graph", data="mixture", n=1000, dim=3,
             nbrs=20, precision="fp32"),
        # a small direction set (the angle), every call on new points
        dict(name="angular_20k_d16", kind="graph", data="angular", n=20000, dim=16,
             nbrs=20, precision="auto"),
        # clustered 8-d points by the landmark scheme with the paper's 60 cells
        dict(name="landmark_20k_d8", kind="landmark", data="clusters", n=20000, dim=8,
             nbrs=20, cells=60, precision="auto"),
        # an ordinary high-dimensional set
        dict(name="manifold_50k_d128", kind="graph", data="manifold", n=50000, dim=128,
             nbrs=70, precision="auto"),
        # the headline workload: a million 128-d descriptors, ~70 neighbours
        dict(name="manifold_1m_d128", kind="graph", data="manifold", n=1000000, dim=128,
             nbrs=70, precision="auto"),
        # the same tree asked again at a wider radius, ~500 neighbours
        dict(name="requery_1m_d128_500", kind="requery", data="manifold", n=1000000,
             dim=128, nbrs=500, precision="auto"),
        # 100K new points against the million kept ones
        dict(name="query_100k_1m_d128", kind="query", data="manifold", n=1000000,
             queries=100000, dim=128, nbrs=70, precision="auto"),
        # an odd, ragged mid-sized table (55 columns, clustered), default
        # precision (direct differences)
        dict(name="table_581012_d55", kind="graph", data="mixture", n=581012, dim=55,
             nbrs=97, precision="fp32"),
        # binary descriptors, 256 bits, an odd count
        dict(name="codes_988258_b256", kind="graph", data="codes", n=988258, dim=256,
             eps=24.0, precision="auto"),
        # edit distance over families of strings
        dict(name="strings_50k", kind="graph", data="strings", n=50000, dim=128,
             eps=6.0, alphabet=4, precision="auto"),
        # many clouds of very different sizes in one forest
        dict(name="clouds_64_d16", kind="batch", data="mixture", clouds=64, lo=1000,
             hi=200000, dim=16, precision="auto"),
        # the cost model over the trace of a million-point query
        dict(name="model_1m", kind="model", n=1000000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["mixture", "manifold", "manifold", "angular", "codes", "strings",
                       "requery", "query", "batch", "landmark", "model"])
    prec = rng.choice(["auto", "auto", "fp32"])
    if kind == "mixture":
        return dict(kind="graph", data="mixture", n=_log(rng, 1000, 600000),
                    dim=rng.randint(2, 78), nbrs=_log(rng, 10, 100), precision=prec)
    if kind == "manifold":
        n = _log(rng, 20000, 1000000)
        return dict(kind="graph", data="manifold", n=n, dim=rng.randint(64, 128),
                    nbrs=_log(rng, 30, 300), precision="auto")
    if kind == "angular":
        return dict(kind="graph", data="angular", n=_log(rng, 1000, 200000),
                    dim=rng.randint(8, 100), nbrs=_log(rng, 10, 100), precision=prec)
    if kind == "codes":
        bits = rng.choice([64, 128, 256, 256, 512])
        n = _log(rng, 10000, 1000000 if bits <= 256 else 300000)
        return dict(kind="graph", data="codes", n=n, dim=bits,
                    eps=float(max(2, bits * 24 // 256)), precision="auto")
    if kind == "strings":
        return dict(kind="graph", data="strings", n=_log(rng, 1000, 80000),
                    dim=rng.choice([64, 100, 128, 200]), eps=float(rng.randint(3, 8)),
                    alphabet=rng.choice([4, 4, 20]), precision="auto")
    if kind == "requery":
        return dict(kind="requery", data="manifold", n=_log(rng, 20000, 1000000),
                    dim=rng.randint(64, 128), nbrs=_log(rng, 30, 500), precision="auto")
    if kind == "query":
        n = _log(rng, 10000, 1000000)
        return dict(kind="query", data=rng.choice(["manifold", "clusters"]), n=n,
                    queries=_log(rng, 100, 100000), dim=rng.randint(8, 128),
                    nbrs=_log(rng, 10, 100), precision="auto")
    if kind == "batch":
        return dict(kind="batch", data="mixture", clouds=_log(rng, 4, 96), lo=1000,
                    hi=_log(rng, 4000, 200000), dim=rng.choice([3, 16, 64]),
                    precision=prec)
    if kind == "landmark":
        return dict(kind="landmark", data="clusters", n=_log(rng, 2000, 70000),
                    dim=rng.randint(4, 32), nbrs=_log(rng, 10, 50),
                    cells=rng.randint(4, 60), precision="auto")
    return dict(kind="model", n=_log(rng, 1000, 4000000))


# ---------------------------------------------------------------- inputs --

class _Rng:
    """Device draws from one seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed) & 0x7FFFFFFF)

    def u(self, lo, hi, *shape):
        return torch.rand(*shape, generator=self.g, device="cuda") * (hi - lo) + lo

    def n(self, *shape):
        return torch.randn(*shape, generator=self.g, device="cuda")

    def i(self, lo, hi, *shape):
        return torch.randint(lo, hi, shape, generator=self.g, device="cuda")


def _mixture(r, n, dim, k):
    """k components, means U[0,1]^dim, sigma log-uniform in [0.01, 0.05]."""
    means = r.u(0.0, 1.0, k, dim)
    sig = torch.exp(r.u(math.log(0.01), math.log(0.05), k))
    lab = r.i(0, k, n)
    return (means[lab] + sig[lab, None] * r.n(n, dim)).contiguous()


def _vectors(r, data, n, dim):
    if data == "mixture":
        return _mixture(r, n, dim, int(r.i(5, 51, 1)[0]))
    if data == "clusters":
        # 20 isotropic clusters of one width
        c = r.u(0.0, 1.0, 20, dim)
        return (c[r.i(0, 20, n)] + 0.05 * r.n(n, dim)).contiguous()
    if data == "angular":
        # directions around 20 unit vectors, random positive lengths
        c = r.n(20, dim)
        c = c / c.norm(dim=1, keepdim=True)
        x = c[r.i(0, 20, n)] + 0.15 * r.n(n, dim)
        return (x * r.u(0.5, 2.0, n, 1)).contiguous()
    # manifold: 12 uniform latents through a random two-layer tanh map
    w1, b1 = r.n(12, 64) * math.sqrt(1 / 12), r.n(64) * 0.1
    w2 = r.n(64, dim) * math.sqrt(1 / 64)
    h = torch.tanh(r.u(-1.0, 1.0, n, 12) @ w1 + b1)
    return (torch.tanh(h @ w2) + 0.01 * r.n(n, dim)).contiguous()


def _centers(case):
    """Codes and strings come in families: this many."""
    return max(8, case["n"] // (244 if case["data"] == "codes" else 50))


def _codes(r, case):
    n, words, k = case["n"], case["dim"] // 64, _centers(case)
    cent = r.i(-2 ** 62, 2 ** 62, k, words) ^ (r.i(0, 2, k, words) << 63)
    lab = torch.arange(n, device="cuda") % k
    out = cent[lab]
    bit = torch.ones(64, dtype=torch.int64, device="cuda") << torch.arange(64, device="cuda")
    for w in range(words):
        for s in range(0, n, 1 << 18):
            m = min(1 << 18, n - s)
            flip = (r.u(0.0, 1.0, m, 64) < 0.05).to(torch.int64)
            out[s:s + m, w] ^= (flip * bit).sum(1)
    return out.contiguous()


def _strings(r, case):
    """Copies of seed strings; each symbol is edited with probability 0.03
    (substituted, preceded by an inserted one, or deleted)."""
    n, stride, a, k = case["n"], case["dim"], case["alphabet"], _centers(case)
    lo, hi = int(stride * 0.625), int(stride * 0.9375)
    length = r.i(lo, hi + 1, k)
    seeds = r.i(0, a, k, hi)
    lab = torch.arange(n, device="cuda") % k
    src, ln = seeds[lab], length[lab]
    hit = r.u(0.0, 1.0, n, hi) < 0.03
    op = r.i(0, 3, n, hi)
    sub = (src + r.i(1, a, n, hi)) % a
    ins = r.i(0, a, n, hi)
    inside = torch.arange(hi, device="cuda")[None, :] < ln[:, None]
    # two slots a position: the inserted symbol, then the symbol itself
    sym = torch.stack([ins, torch.where(hit & (op == 0), sub, src)], 2).view(n, 2 * hi)
    keep = torch.stack([inside & hit & (op == 1), inside & ~(hit & (op == 2))], 2)
    keep = keep.view(n, 2 * hi)
    pos = torch.cumsum(keep, 1) - 1
    keep &= pos < stride
    out = torch.full((n, stride + 1), 0xFF, dtype=torch.uint8, device="cuda")
    out.scatter_(1, torch.where(keep, pos, stride), torch.where(keep, sym, 255).to(torch.uint8))
    return out[:, :stride].contiguous()


def _rows_dist(metric, q, x):
    """Distances of rows q to all rows x in 64 bits."""
    q, x = q.double(), x.double()
    if metric == "angular":
        q, x = q / q.norm(dim=1, keepdim=True), x / x.norm(dim=1, keepdim=True)
    d = torch.empty(q.shape[0], x.shape[0], dtype=torch.float64, device="cuda")
    for i in range(q.shape[0]):
        d[i] = (x - q[i]).square().sum(1).sqrt()
    return 2 * torch.asin((d / 2).clamp(max=1)) if metric == "angular" else d


def _radius(metric, x, nbrs, queries=None):
    """The radius that gives sampled rows `nbrs` neighbours on average, to
    five digits."""
    src = x if queries is None else queries
    rows = min(src.shape[0], 64 if x.shape[0] > 4000 else 128)
    at = torch.linspace(0, src.shape[0] - 1, rows, device="cuda").long()
    d = _rows_dist(metric, src[at], x)
    if queries is None:
        d[torch.arange(rows, device="cuda"), at] = math.inf
    k = max(1, min(int(nbrs * rows), d.numel() - rows - 1))
    v = torch.topk(d.flatten(), k + 1, largest=False).values
    return float("%.5g" % float((v[k - 1] + v[k]) / 2))


def _metric(case):
    return {"angular": "angular", "codes": "hamming", "strings": "levenshtein"}.get(
        case.get("data"), "l2")


def _model_inputs(case, seed):
    r = _Rng(seed)
    x = r.n(case["n"], 16).contiguous()
    # targets: log counts that depend on the features, with noise
    t = torch.stack([3 + x[:, 0] * x[:, 1], 4 + torch.sin(x[:, 2]) + 0.3 * x[:, 3]], 1)
    t = (t + 0.2 * r.n(case["n"], 2)).contiguous()
    p = [r.n(*s) * math.sqrt(1 / s[1]) if len(s) == 2 else 0.1 * r.n(*s) for s in MLP_SHAPES]
    return torch.cat([q.flatten() for q in p]).contiguous(), x, t


def _axes(r, xs):
    """One pose for vectors that share their axes: axes reordered, some
    mirrored, each set's rows reordered."""
    dim = xs[0].shape[1]
    order, sign = torch.argsort(r.u(0, 1, dim)), 1.0 - 2.0 * r.i(0, 2, dim)
    return [(x[torch.argsort(r.u(0, 1, x.shape[0]))][:, order] * sign).contiguous()
            for x in xs]


def _inputs(case, seed):
    """Points, per-cloud offsets (None for one set), radius or radii, queries."""
    key = zlib.crc32(repr(sorted((k, v) for k, v in case.items() if k != "name")).encode())
    r, pose = _Rng(key), _Rng(seed)
    data = case["data"]
    if case["kind"] == "batch":
        h = np.random.default_rng(key)
        ns = np.exp(h.uniform(math.log(case["lo"]), math.log(case["hi"]), case["clouds"]))
        ns = np.rint(ns).astype(np.int64)
        want = np.exp(h.uniform(math.log(10), math.log(300), case["clouds"]))
        comps = h.integers(5, 51, case["clouds"])
        xs = [_mixture(r, int(n), case["dim"], int(k)) for n, k in zip(ns, comps)]
        eps = [_radius("l2", x, min(w, 0.2 * len(x))) for x, w in zip(xs, want)]
        at = np.random.default_rng(int(seed)).permutation(len(xs))
        xs, eps = _axes(pose, [xs[i] for i in at]), [eps[i] for i in at]
        return torch.cat(xs), np.concatenate([[0], np.cumsum(ns[at])]), eps, None
    if data in ("codes", "strings"):
        x = _codes(r, case) if data == "codes" else _strings(r, case)
        x = x[torch.argsort(pose.u(0, 1, x.shape[0]))]
        if data == "codes":
            x = x[:, torch.argsort(pose.u(0, 1, x.shape[1]))] ^ pose.i(-2 ** 62, 2 ** 62,
                                                                        x.shape[1])
        else:
            name = torch.full((256,), 0xFF, dtype=torch.uint8, device="cuda")
            name[:case["alphabet"]] = torch.argsort(pose.u(0, 1, case["alphabet"])).to(
                torch.uint8)
            x = name[x.long()]
        return x.contiguous(), None, case["eps"], None
    nq = case.get("queries", 0)
    x = _vectors(r, data, case["n"] + nq, case["dim"])
    x, q = x[:case["n"]], x[case["n"]:] if nq else None
    eps = _radius(_metric(case), x, case["nbrs"], q)
    xs = _axes(pose, [x, q] if nq else [x])
    return xs[0], None, eps, xs[1] if nq else None


def prepare(case, seed):
    if case["kind"] == "model":
        p, x, t = _model_inputs(case, seed)
        return {"kind": "model", "params": p, "x": x, "t": t}
    x, off, eps, q = _inputs(case, seed)
    st = {"kind": case["kind"], "metric": _metric(case), "x": x, "offsets": off, "eps": eps,
          "q": q, "precision": case["precision"], "cells": case.get("cells", 0)}
    if case["kind"] in ("requery", "query"):
        st["tree"] = fnn.fnn_tree_build(x, st["metric"])
    return st


def run(state):
    s = state
    if s["kind"] == "model":
        y = fnn.fnn_mlp_forward(s["params"], s["x"])
        loss, grad = fnn.fnn_mlp_loss_grad(s["params"], s["x"], s["t"])
        return {"y": y, "loss": loss, "grad": grad}
    if s["kind"] == "landmark":
        g = fnn.fnn_landmark_eps_graph(s["x"], s["eps"], s["cells"], s["metric"],
                                       precision=s["precision"])
    elif s["kind"] == "query":
        g = fnn.fnn_eps_query(s["tree"], s["q"], s["eps"], precision=s["precision"])
    elif s["kind"] == "batch":
        tree = fnn.fnn_tree_build_batch(s["x"], s["offsets"], s["metric"])
        g = fnn.fnn_eps_graph_batch(tree, s["eps"], precision=s["precision"])
    else:
        tree = s["tree"] if s["kind"] == "requery" else fnn.fnn_tree_build(s["x"], s["metric"])
        g = fnn.fnn_eps_graph(tree, s["eps"], precision=s["precision"])
    return {"row_ptr": g.row_ptr, "col": g.col, "dist": g.dist}


def work(case):
    if case["kind"] == "model":
        # inputs and targets once, predictions once; 2 ops a weight and
        # sample for each of two forward passes, 4 for the backward one
        n, w = case["n"], sum(a * b for a, b in (s for s in MLP_SHAPES if len(s) == 2))
        return {"bytes": 4.0 * n * (16 + 2 + 2), "flops": float(n) * 8 * w}
    if case["kind"] == "batch":
        # sizes are log-uniform, mean neighbour counts log-uniform in 10..300
        lo, hi = case["lo"], case["hi"]
        n = case["clouds"] * (hi - lo) / max(math.log(hi / lo), 1e-9) if hi > lo else (
            case["clouds"] * lo)
        nbrs = 290 / math.log(30)
    else:
        n = case["n"]
        nbrs = case.get("nbrs")
    d = case["dim"]
    if case["data"] == "codes":
        # about half of a family lies within the radius
        row, ops, nbrs = d / 8, d / 32, 0.5 * n / _centers(case)
    elif case["data"] == "strings":
        row, ops, nbrs = d, 4.0 * d, 0.6 * n / _centers(case)
    else:
        row, ops = 4.0 * d, 3.0 * d
    out = case.get("queries", n)
    nnz = out * nbrs
    pairs = nnz if case.get("queries") else nnz / 2
    return {"bytes": n * row + case.get("queries", 0) * row + 8.0 * nnz + 8.0 * out,
            "flops": pairs * ops}


# ------------------------------------------------- the same in 64 bits --

def _csr(counts, cols, dists):
    rp = torch.zeros(sum(c.numel() for c in counts) + 1, dtype=torch.int64, device="cuda")
    rp[1:] = torch.cumsum(torch.cat(counts), 0)
    return {"row_ptr": rp, "col": torch.cat(cols).to(torch.int32), "dist": torch.cat(dists)}


def _exact_vectors(metric, x, eps, q=None):
    """Rows of q (or x, without the pairs of a row with itself) against x:
    counts per row, columns, distances."""
    x = x.double()
    q = x if q is None else q.double()
    same = q is x
    if metric == "angular":
        x = x / x.norm(dim=1, keepdim=True)
        q = x if same else q / q.norm(dim=1, keepdim=True)
    r2 = (2 * math.sin(min(eps, math.pi) / 2)) ** 2 if metric == "angular" else eps * eps
    # a float32 screen of |a|^2 + |b|^2 - 2ab with room for its rounding, then
    # the direct difference in 64 bits
    mu = x.mean(0)
    xf, qf = (x - mu).float(), (q - mu).float()
    hx, hq = xf.square().sum(1) / 2, qf.square().sum(1) / 2
    room = 2e-7 * (x.shape[1] + 16) * float(torch.maximum(hx.max(), hq.max()))
    xt = xf.t().contiguous()
    counts, cols, dists = [], [], []
    step = max(1, min(q.shape[0], 1_000_000_000 // x.shape[0]))
    for s in range(0, q.shape[0], step):
        e = min(q.shape[0], s + step)
        near = torch.addmm(hx, qf[s:e], xt, beta=-1) >= (hq[s:e] - r2 / 2 - room)[:, None]
        i, j = near.nonzero(as_tuple=True)
        del near
        i = i + s
        if same:
            keep = i != j
            i, j = i[keep], j[keep]
        d = torch.empty(i.numel(), dtype=torch.float64, device="cuda")
        for b in range(0, i.numel(), 1 << 21):
            a, c = q[i[b:b + (1 << 21)]], x[j[b:b + (1 << 21)]]
            t = (a - c).square().sum(1).sqrt()
            if metric == "angular":
                t = 2 * torch.atan2(t, (a + c).square().sum(1).sqrt())
            d[b:b + (1 << 21)] = t
        keep = d <= eps
        counts.append(torch.bincount(i[keep] - s, minlength=e - s))
        cols.append(j[keep].to(torch.int32))
        dists.append(d[keep])
    return counts, cols, dists


def _exact_codes(x, eps):
    n, words = x.shape
    bits = words * 64
    k = int(math.floor(eps))
    s = torch.arange(64, device="cuda")
    pm = torch.cat([(((x[:, w, None] >> s) & 1) * 2 - 1).half() for w in range(words)], 1)
    pt = pm.t().contiguous()
    counts, cols, dists = [], [], []
    step = max(1, min(n, 1_000_000_000 // n))
    for b in range(0, n, step):
        g = pm[b:b + step] @ pt                       # bits - 2 distance, whole
        i, j = (g >= bits - 2 * k).nonzero(as_tuple=True)
        keep = i + b != j
        i, j = i[keep], j[keep]
        counts.append(torch.bincount(i, minlength=min(step, n - b)))
        cols.append(j.to(torch.int32))
        dists.append((bits - g[i, j].double()) / 2)
    return counts, cols, dists


def _edit(a, b, la, lb, k):
    """Edit distances of string pairs inside a band of k (beyond it: more
    than k)."""
    far, width = 99, 2 * k + 1
    p, size = a.shape
    full = lambda v: torch.full((p,), v, dtype=torch.int16, device="cuda")  # noqa: E731
    prev = [full(c - k if c >= k else far) for c in range(width)]
    res = full(far)
    end = (lb - la + k).clamp(0, 2 * k)
    for i in range(size + 1):
        if i:
            cur = []
            for c in range(width):
                j = i + c - k
                if j < 0 or j > size:
                    cur.append(full(far))
                elif j == 0:
                    cur.append(full(i))
                else:
                    v = prev[c] + (a[:, i - 1] != b[:, j - 1]).to(torch.int16)
                    if c + 1 < width:
                        v = torch.minimum(v, prev[c + 1] + 1)
                    if c:
                        v = torch.minimum(v, cur[c - 1] + 1)
                    cur.append(v)
            prev = cur
        at = (la == i).nonzero().flatten()
        if at.numel():
            rows = torch.stack([c[at] for c in prev], 1)
            res[at] = rows.gather(1, end[at, None])[:, 0]
    return torch.where((la - lb).abs() > k, far, res)


def _exact_strings(x, eps, alphabet):
    """Pairs whose counts of three-symbol runs differ by at most 6 an edit
    (an edit removes and adds at most three), then the edit distance."""
    n, k = x.shape[0], int(math.floor(eps))
    ln = (x != 0xFF).sum(1)
    v = x.long()
    gram = ((v[:, :-2] * alphabet + v[:, 1:-1]) * alphabet + v[:, 2:]) % 61
    ok = torch.arange(gram.shape[1], device="cuda")[None, :] + 2 < ln[:, None]
    cnt = torch.zeros(n, 62, device="cuda")
    cnt.scatter_add_(1, torch.where(ok, gram, 61), torch.ones_like(gram, dtype=torch.float32))
    cnt[:, 61] = 0
    top = int(cnt.max())
    # min(a, b) = sum over t of [a >= t][b >= t], a product of zeros and ones
    steps = torch.cat([(cnt >= t).half() for t in range(1, top + 1)], 1)
    st, size = steps.t().contiguous(), cnt.sum(1)
    counts, cols, dists = [], [], []
    rows = max(1, min(n, 400_000_000 // n))
    for s in range(0, n, rows):
        e = min(n, s + rows)
        both = (steps[s:e] @ st).float()
        i, j = (size[s:e, None] + size - 2 * both <= 6 * k).nonzero(as_tuple=True)
        i = i + s
        keep = (i != j) & ((ln[i] - ln[j]).abs() <= k)
        i, j = i[keep], j[keep]
        d = torch.cat([_edit(x[i[b:b + (1 << 21)]], x[j[b:b + (1 << 21)]],
                             ln[i[b:b + (1 << 21)]], ln[j[b:b + (1 << 21)]], k)
                       for b in range(0, max(1, i.numel()), 1 << 21)])
        keep = d <= k
        counts.append(torch.bincount(i[keep] - s, minlength=e - s))
        cols.append(j[keep].to(torch.int32))
        dists.append(d[keep].double())
    return counts, cols, dists


def _exact_model(p, x, t):
    w, at = [], 0
    for s in MLP_SHAPES:
        m = math.prod(s)
        w.append(p[at:at + m].double().view(*s).requires_grad_())
        at += m
    y, loss = [], 0.0
    for b in range(0, x.shape[0], 1 << 20):
        h = torch.nn.functional.silu(x[b:b + (1 << 20)].double() @ w[0].t() + w[1])
        h = torch.nn.functional.silu(h @ w[2].t() + w[3])
        o = h @ w[4].t() + w[5]
        part = (o - t[b:b + (1 << 20)].double()).square().sum() / (2 * x.shape[0])
        part.backward()
        loss += float(part.detach())
        y.append(o.detach())
    return {"y": torch.cat(y), "loss": loss, "grad": torch.cat([v.grad.flatten() for v in w])}


def exact(case, seed):
    if case["kind"] == "model":
        return _exact_model(*_model_inputs(case, seed))
    x, off, eps, q = _inputs(case, seed)
    if case["data"] == "codes":
        return _csr(*_exact_codes(x, eps))
    if case["data"] == "strings":
        return _csr(*_exact_strings(x, eps, case["alphabet"]))
    if off is None:
        return _csr(*_exact_vectors(_metric(case), x, eps, q))
    counts, cols, dists = [], [], []
    for c, e in enumerate(eps):
        a, b, d = _exact_vectors("l2", x[off[c]:off[c + 1]], e)
        counts, dists = counts + a, dists + d
        cols += [j + int(off[c]) for j in b]
    return _csr(counts, cols, dists)

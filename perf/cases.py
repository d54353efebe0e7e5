"""The work that users of this library have it do, as cases that can be timed and compared.

A case is one of three tasks:

  epoch   ``Som.train_epoch``: one epoch at some point of a cooled schedule, from the code book that the
          schedule has reached there, on the registered training set (what a long run consists of) or on a
          batch that is not registered (a stream), under any of the neighbourhood functions;
  train   ``Som.train``: a whole schedule on a small table, registration included;
  place   the use of a trained map: BMUs of new instances, their distances to them and the mean
          quantisation error, and the U-matrix where the whole data set is mapped after training.

Data are dense mixtures or uniform noise, sparse text-like rows (Zipf columns), or sparse uniform rows, with
the recipes of ``gen/workloads.py`` redrawn on the GPU.  Larger runs are timed an epoch at a time, because
a whole schedule amplifies the last bits of its sums (an instance between two nearly equal nodes moves from
one to the other), so that only its early epochs could be compared.
"""
from __future__ import annotations

import math

import torch

from paper_1305_1422_amd import Som, capi

DEV = "cuda:0"


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # a first run on a small table: every launch counts (configuration 1 of the benchmark)
        dict(name="toy_train", task="train", data="uniform", n=1_000, dim=10, rows=20, cols=20, map="planar",
             grid="square", neighborhood="gaussian", compact=False, epochs=10),
        # serving: a handful of new instances against a trained map of the common size
        dict(name="place_few", task="place", data="mixture", n=64, dim=1_000, rows=50, cols=50, map="toroid",
             grid="square", components=16, sigma=0.05, umatrix=False),
        # a batch of a stream that is not registered, odd in every size, on a planar hexagonal map
        dict(name="stream_epoch", task="epoch", data="mixture", n=4_097, dim=33, rows=37, cols=29, map="planar",
             grid="hexagonal", neighborhood="gaussian", compact=False, components=24, sigma=0.1, progress=0.5,
             registered=False),
        # new documents placed on a trained text map
        dict(name="place_text", task="place", data="zipf", n=1_000, dim=50_000, rows=50, cols=50, map="planar",
             grid="square", umatrix=False),
        # the other neighbourhood function, ordinary table, ragged sizes
        dict(name="bubble_epoch", task="epoch", data="mixture", n=20_011, dim=100, rows=45, cols=60, map="toroid",
             grid="hexagonal", neighborhood="bubble", compact=False, components=40, sigma=0.1, progress=0.5,
             registered=True),
        # the data set mapped onto the trained map, with its quality figures (configuration 2's shape)
        dict(name="place_all", task="place", data="mixture", n=100_000, dim=1_000, rows=50, cols=50, map="toroid",
             grid="square", components=16, sigma=0.05, umatrix=True),
        # the headline training run, in the middle of its schedule (configuration 2)
        dict(name="dense_epoch", task="epoch", data="mixture", n=100_000, dim=1_000, rows=50, cols=50, map="toroid",
             grid="square", neighborhood="gaussian", compact=False, components=16, sigma=0.05, progress=0.5,
             registered=True),
        # an emergent map, about as many nodes as instances, late in its schedule (configuration 3)
        dict(name="emergent_epoch", task="epoch", data="mixture", n=50_000, dim=256, rows=200, cols=200, map="toroid",
             grid="hexagonal", neighborhood="gaussian", compact=False, components=64, sigma=0.1, progress=0.75,
             registered=True),
        # many instances of few features, early in the schedule (configuration 5)
        dict(name="large_epoch", task="epoch", data="mixture", n=1_000_000, dim=128, rows=100, cols=100, map="planar",
             grid="hexagonal", neighborhood="gaussian", compact=False, components=256, sigma=0.03, progress=0.25,
             registered=True),
        # text-like sparse rows (configuration 4)
        dict(name="text_epoch", task="epoch", data="zipf", n=100_000, dim=50_000, rows=50, cols=50, map="planar",
             grid="square", neighborhood="gaussian", compact=False, progress=0.5, registered=True),
        # random sparse rows of modest dimension, the last epoch (configuration 6)
        dict(name="sparse_epoch", task="epoch", data="sparse_uniform", n=100_000, dim=1_000, rows=50, cols=50,
             map="planar", grid="square", neighborhood="gaussian", compact=False, density=0.05, progress=1.0,
             registered=True),
        # the emergent text map: more nodes than documents (configuration 7)
        dict(name="text_esom_epoch", task="epoch", data="zipf", n=12_347, dim=20_000, rows=205, cols=336, map="toroid",
             grid="square", neighborhood="gaussian", compact=False, progress=0.5, registered=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: a task, a kind of data and sizes from the ranges that the listed cases span."""
    kind = rng.choice(["epoch dense", "epoch dense", "epoch dense", "epoch zipf", "epoch uniform", "train",
                       "place dense", "place zipf"])
    task, dense = kind.split()[0], kind in ("epoch dense", "train", "place dense")
    while True:
        c = dict(task=task, map=rng.choice(["planar", "toroid"]), grid=rng.choice(["square", "hexagonal"]))
        if kind == "train":
            c.update(n=_log_int(rng, 200, 5_000), dim=_log_int(rng, 3, 40), rows=rng.randint(8, 24), epochs=rng.randint(5, 10))
        elif task == "epoch":
            c.update(n=_log_int(rng, 1_000, 1_000_000 if dense else 100_000), rows=_log_int(rng, 10, 200),
                     progress=round(rng.random(), 3), registered=rng.random() < 0.7)
        else:
            c.update(n=_log_int(rng, 1, 100_000 if dense else 20_000), rows=_log_int(rng, 10, 80),
                     umatrix=rng.random() < 0.5)
        if dense:
            c.update(data=rng.choice(["mixture", "mixture", "uniform"]), components=rng.randint(8, 256),
                     sigma=round(math.exp(rng.uniform(math.log(0.03), math.log(0.15))), 4))
            c.setdefault("dim", _log_int(rng, 3, 1_200))
        elif kind == "epoch uniform":
            c.update(data="sparse_uniform", dim=_log_int(rng, 200, 1_500), density=round(rng.uniform(0.02, 0.08), 3))
        else:
            c.update(data="zipf", dim=_log_int(rng, 5_000, 50_000))
        c["cols"] = max(8, int(c["rows"] * rng.uniform(0.7, 1.6)))
        if task != "place":
            other = dense and rng.random() < 0.25
            c.update(neighborhood=rng.choice(["gaussian", "bubble"]) if other else "gaussian", compact=other)
        k = c["rows"] * c["cols"]
        if work(c)["flops"] > 2.6e12 or k > 40_000 or k * c["dim"] > 1.3e8 or (dense and c["n"] * c["dim"] > 1.3e8):
            continue
        if task == "place" and k > 6_400:
            continue
        return c


# ---------------------------------------------------------------- data
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _rand(g, *shape):
    return torch.rand(shape, generator=g, device=DEV, dtype=torch.float32)


def _dense(case, g, n, means):
    if case["data"] == "uniform":
        return _rand(g, n, case["dim"])
    which = torch.randint(means.shape[0], (n,), generator=g, device=DEV)
    x = torch.randn((n, case["dim"]), generator=g, device=DEV, dtype=torch.float32)
    return x.mul_(case["sigma"]).add_(means[which])


def _zipf_rows(g, n, dim, mean_len=100.0, max_len=400, s=1.1, lam=2.0):
    """Row lengths Poisson(mean_len) in [1, max_len]; the first so many distinct columns of a sequence of Zipf
    draws, sorted; values log(2 + Poisson(lam)), rows of unit length."""
    cdf = torch.cumsum(torch.arange(1, dim + 1, device=DEV, dtype=torch.float64) ** -s, 0)
    cdf = (cdf / cdf[-1]).float()
    parts = []
    for at in range(0, n, 20_000):
        m = min(20_000, n - at)
        lens = torch.poisson(torch.full((m,), mean_len, device=DEV), generator=g).clamp_(1, min(max_len, dim))
        cols = torch.searchsorted(cdf, _rand(g, m, 768), right=True).clamp_(max=dim - 1)
        ordered, pos = torch.sort(cols, dim=1, stable=True)
        first = torch.ones_like(ordered, dtype=torch.bool)
        first[:, 1:] = ordered[:, 1:] != ordered[:, :-1]
        drawn = torch.zeros_like(first).scatter_(1, pos, first)      # in draw order: is it a new column?
        rank = torch.cumsum(drawn, 1).gather(1, pos)                 # of every sorted entry: how many distinct so far
        keep = first & (rank <= lens[:, None])
        v = torch.log(2.0 + torch.poisson(torch.full(cols.shape, lam, device=DEV), generator=g)) * keep
        v = v / v.square().sum(1, keepdim=True).sqrt()
        parts.append((keep.sum(1), ordered[keep].int(), v[keep].float()))
    indptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    indptr[1:] = torch.cumsum(torch.cat([p[0] for p in parts]), 0)
    return indptr, torch.cat([p[1] for p in parts]), torch.cat([p[2] for p in parts])


def _uniform_rows(g, n, dim, density):
    """Every entry nonzero with the given probability, values uniform [0, 1)."""
    counts, cols = [], []
    step = max(1, (1 << 26) // dim)
    for at in range(0, n, step):
        hit = _rand(g, min(step, n - at), dim) < density
        counts.append(hit.sum(1))
        cols.append(hit.nonzero()[:, 1].int())
    indptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    indptr[1:] = torch.cumsum(torch.cat(counts), 0)
    cols = torch.cat(cols)
    return indptr, cols, _rand(g, cols.numel())


def _rows(case, g, n, means):
    if case["data"] == "zipf":
        return _zipf_rows(g, n, case["dim"])
    if case["data"] == "sparse_uniform":
        return _uniform_rows(g, n, case["dim"], case["density"])
    return _dense(case, g, n, means)


def _densified(csr, dim):
    n = csr[0].numel() - 1
    row = torch.repeat_interleave(torch.arange(n, device=DEV), csr[0].diff())
    out = torch.zeros((n, dim), device=DEV)
    out[row, csr[1].long()] = csr[2]
    return out


def _grid_sq(case, chosen):
    """Squared grid distance of every node to the chosen ones."""
    rows, cols, hexa = case["rows"], case["cols"], case["grid"] == "hexagonal"
    y = torch.arange(rows, device=DEV).repeat_interleave(cols)
    x2 = 2 * torch.arange(cols, device=DEV).repeat(rows) + (y % 2 if hexa else 0)
    dy, dx = (y[:, None] - y[chosen]).abs(), (x2[:, None] - x2[chosen]).abs()
    if case["map"] == "toroid":
        dy, dx = torch.minimum(dy, rows - dy), torch.minimum(dx, (2 * cols - dx).abs())
    return dx.float().square() / 4 + dy.float().square() * (0.75 if hexa else 1.0)


def _radius(case, progress):
    r0 = max(1.0, min(case["rows"], case["cols"]) / 2)
    return r0 + (1.0 - r0) * progress


def _trained(case, x, w, epochs, progress):
    """The code book that the plain batch rule reaches on a sample, the radius cooled as far as `progress`."""
    for e in range(epochs):
        r = _radius(case, progress * e / (epochs - 1))
        q = _grid_sq(case, torch.argmin(w.square().sum(1) - 2 * (x @ w.T), 1))
        h = torch.exp(q / (-2 * r * r)) if case.get("neighborhood", "gaussian") == "gaussian" else (q <= r * r).float()
        if case.get("compact"):
            h = h * (q <= r * r)
        mass = h.sum(1, keepdim=True)
        w = torch.where(mass > 1e-20, (h @ x) / mass.clamp_min(1e-20), w)
    return w.contiguous()


# ---------------------------------------------------------------- a pass
def prepare(case, seed):
    g = _gen(seed)
    k, dim = case["rows"] * case["cols"], case["dim"]
    means = _rand(g, int(case.get("components", 1)), dim)
    w0 = _rand(g, k, dim)
    data = _rows(case, g, case["n"], means)
    if case["task"] != "train":
        sample = _rows(case, g, 4_096 if k * dim < 2e8 else 2_048, means)
        if isinstance(sample, tuple):
            sample = _densified(sample, dim)
        if case["task"] == "place":
            w0 = _trained(case, sample, w0, 8, 1.0)
        else:      # the code book that enters the epoch left the one before it, of a schedule of ten
            w0 = _trained(case, sample, w0, 4, max(0.0, case["progress"] - 1 / 9))
        del sample
    som = Som(case["rows"], case["cols"], dim, case["map"], case["grid"], codebook=w0)
    if case.get("neighborhood", "gaussian") != "gaussian" or case.get("compact"):
        som.set_neighborhood(case["neighborhood"], case["compact"])
    if case.get("registered"):
        if isinstance(data, tuple):
            capi.som_set_data_csr(som.ctx, *data)
        else:
            capi.som_set_data_dense(som.ctx, data)
    return dict(case=case, data=data, som=som, w0=w0)


def run(state):
    case, som, data = state["case"], state["som"], state["data"]
    if case["task"] == "place":
        bmus = som.bmus(data)
        dist, qerror = som.bmu_distances(data, bmus)
        out = {"bmus": bmus, "distances": dist, "qerror": qerror}
        if case["umatrix"]:
            out["umatrix"] = som.umatrix()
        return out
    som.codebook.copy_(state["w0"])
    if case["task"] == "train":
        bmus = som.train(data, case["epochs"])
    else:
        bmus = som.train_epoch(data, _radius(case, case["progress"]))
    return {"bmus": bmus, "codebook": som.codebook}


# ---------------------------------------------------------------- what a pass cannot do without
def _nonzeros(case):
    if case["data"] == "zipf":
        return 100.0 * case["n"]
    if case["data"] == "sparse_uniform":
        return case["density"] * case["n"] * case["dim"]
    return float(case["n"]) * case["dim"]


def _search_flops(case):
    """One multiply-add per nonzero and node."""
    return 2.0 * _nonzeros(case) * case["rows"] * case["cols"]


def work(case):
    n, dim, k, nnz = case["n"], case["dim"], case["rows"] * case["cols"], _nonzeros(case)
    sparse = case["data"] in ("zipf", "sparse_uniform")
    data_bytes = nnz * 8 + (n + 1) * 8 if sparse else nnz * 4
    if case["task"] == "place":
        # data and code book in; BMUs, distances, mean (and U-matrix) out
        return {"bytes": data_bytes + 4.0 * k * dim + 8.0 * n + 8 + (4.0 * k if case["umatrix"] else 0),
                "flops": _search_flops(case) + 2 * nnz + (6.0 * k * dim if case["umatrix"] else 0)}
    # data and code book in, code book and BMUs out; a search, the sums and the separable smoothing per epoch (the last
    # for any neighbourhood: at least one multiply-add per node and channel)
    smooth = 2.0 * k * dim * (case["rows"] + case["cols"] if case["neighborhood"] == "gaussian" and not case["compact"] else 1)
    return {"bytes": data_bytes + 8.0 * k * dim + 4.0 * n,
            "flops": case.get("epochs", 1) * (_search_flops(case) + nnz + smooth)}


def tolerance(case):
    # A search is decided exactly, so its BMUs are the same whatever finds them; distances are rounded once from
    # double sums; a code book is a ratio of 32-bit sums.
    if case["task"] == "place":
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}
    if case["task"] == "epoch":
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.0}
    # a whole schedule: an instance or two may have changed nodes on the way, and its neighbourhood with it
    return {"rel": 1e-3, "max": 0.1, "differ": 0.005}

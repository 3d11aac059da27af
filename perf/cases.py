"""The workloads this library is timed on: its public calls, at the sizes its users run them.

A case is a dict of plain values.  ``kind`` names the call:

* ``dm``      one distance matrix (or one piece of it, as stripes) from an uploaded table
* ``step``    a study from its resident table: scalars, both sparse splits, both matrices
* ``batch``   many rarefied tables on one tree, one graph replay
* ``pcoa``    principal coordinates of a matrix
* ``mantel``  Mantel test of two matrices
* ``train``   steps of encoder training, then the parameters are read out
* ``encode``  projection of new samples and the encoder's forward pass
* ``place``   nearest references in the encoder's space, exact re-rank

``prepare`` makes what a program holds before the call, from the seed alone; ``run`` is one
pass; ``exact`` is the same result in 64 bits by plain torch.
"""
import math

import numpy as np
import torch

import paper_2107_05397_amd as uf
from paper_2107_05397_amd import placement

DEV = "cuda"


# --------------------------------------------------------------------------- cases
def listed():
    return [
        # the smallest study anybody runs: 256 samples x 1,000 tips, 50 of them per sample,
        # in the default precision with the centring terms of an ordination; latency and
        # launches count
        dict(name="dm_smallest", kind="dm", tips=1000, samples=256, nnz=50, law="uniform",
             variant="weighted", precision="fp64", out="f64", means=True, pieces=1),
        # an ordinary study in the default precision of the weighted distance
        dict(name="dm_weighted_fp64", kind="dm", tips=20000, samples=1500, nnz=300, law="zipf",
             variant="weighted", precision="fp64", out="f64", means=False, pieces=1),
        # the same, unweighted, with an odd number of samples and the centring terms
        dict(name="dm_unweighted_fp64", kind="dm", tips=20000, samples=2001, nnz=300, law="zipf",
             variant="unweighted", precision="fp64", out="f64", means=True, pieces=1),
        # a larger study in the default precision of the unweighted distance
        dict(name="dm_unweighted_mfma", kind="dm", tips=100000, samples=5000, nnz=500, law="zipf",
             variant="unweighted", precision="mfma", out="f32", means=False, pieces=1),
        # weighted distances again and again from a kept embedding and its split
        dict(name="dm_weighted_split", kind="dm", tips=50000, samples=3333, nnz=500, law="zipf",
             variant="weighted", precision="fp32_split", out="f32", means=False, pieces=1),
        # the benchmark's step on a fifth of its samples: everything from the resident table
        dict(name="step_both", kind="step", tips=200000, samples=10000, nnz=1000, law="zipf"),
        # rarefied replicates of uneven size on one tree, replayed as one graph
        dict(name="batch_fp32", kind="batch", tips=10000, tables=8, n_min=300, n_max=1500, nnz=300,
             depth=1000, precision="fp32"),
        # ordination of a matrix: ten axes, twenty columns, three passes, as the benchmark runs it
        dict(name="pcoa", kind="pcoa", samples=6000, dims=10, cols=20, iters=3, means=True),
        # Mantel test with the usual 999 permutations
        dict(name="mantel", kind="mantel", samples=2000, perms=999, method="pearson",
             alternative="two-sided"),
        # the placement encoder: training steps of 2,048 triples, then a checkpoint
        dict(name="train", kind="train", rows=8192, d0=4096, hidden=1024, dz=128, triples=2048,
             steps=24),
        # new samples into the encoder's space
        dict(name="encode", kind="encode", tips=100000, samples=3000, nnz=500, d0=4096, hidden=1024,
             dz=128),
        # new samples against a reference set: kNN and the exact re-rank of 100 candidates
        dict(name="place", kind="place", tips=100000, refs=6000, queries=1500, nnz=500, dz=128,
             candidates=100, k=10),
    ]


def _log(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def draw(rng):
    kind = rng.choice(["dm"] * 8 + ["step", "batch", "batch", "pcoa", "pcoa", "mantel", "mantel",
                                    "train", "encode", "place"])
    if kind == "dm":
        variant = rng.choice(["weighted", "unweighted"])
        precision = rng.choice(["fp64", "fp64", "fp32", "fp32_split" if variant == "weighted" else
                                "mfma_split"] + (["mfma"] if variant == "unweighted" else []))
        n, tips = _log(rng, 64, 5000), _log(rng, 500, 100000)
        if precision in ("fp64", "fp32"):   # every pair over every branch on the vector units
            tips = max(500, min(tips, int(2e11 / n / n)))
        return dict(kind="dm", tips=tips, samples=n, nnz=max(5, min(_log(rng, 30, 600), tips // 4)),
                    law=rng.choice(["uniform", "zipf"]), variant=variant, precision=precision,
                    out="f64" if precision == "fp64" else "f32",
                    means=precision == "fp64" and rng.random() < 0.5,
                    pieces=rng.choice([1, 1, 1, 3]))
    if kind == "step":
        return dict(kind="step", tips=_log(rng, 5000, 200000), samples=_log(rng, 300, 10000),
                    nnz=_log(rng, 100, 1000), law="zipf")
    if kind == "batch":
        lo = _log(rng, 60, 800)
        return dict(kind="batch", tips=_log(rng, 1000, 20000), tables=rng.randint(2, 10), n_min=lo,
                    n_max=int(lo * rng.uniform(1.5, 2.5)), nnz=_log(rng, 50, 250),
                    depth=_log(rng, 300, 2000), precision=rng.choice(["fp32", "fp32", "fp32_split"]))
    if kind == "pcoa":
        dims = rng.randint(2, 12)
        return dict(kind="pcoa", samples=_log(rng, 60, 10000), dims=dims, cols=dims + rng.randint(5, 12),
                    iters=rng.randint(1, 4), means=rng.random() < 0.7)
    if kind == "mantel":
        method = rng.choice(["pearson", "spearman"])
        n = _log(rng, 50, 4000)
        return dict(kind="mantel", samples=n, perms=rng.choice([99, 199, 999] if n <= 2000 else [99, 199]),
                    method=method, alternative=rng.choice(["two-sided", "greater", "less"]))
    if kind == "train":
        return dict(kind="train", rows=_log(rng, 1000, 8192), d0=rng.choice([1024, 2048, 4096]),
                    hidden=rng.choice([256, 512, 1024]), dz=rng.choice([64, 96, 128]),
                    triples=_log(rng, 256, 2048), steps=24)
    if kind == "encode":
        return dict(kind="encode", tips=_log(rng, 5000, 100000), samples=_log(rng, 50, 3000),
                    nnz=_log(rng, 50, 500), d0=rng.choice([1024, 2048, 4096]),
                    hidden=rng.choice([256, 512, 1024]), dz=rng.choice([64, 96, 128]))
    return dict(kind="place", tips=_log(rng, 5000, 100000), refs=_log(rng, 500, 6000),
                queries=_log(rng, 20, 1500), nnz=_log(rng, 50, 500), dz=rng.choice([64, 96, 128]),
                candidates=rng.choice([10, 40, 100]), k=10)


# --------------------------------------------------------------------------- inputs
def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1009 + stream)
    return g


def _tree(tips, seed):
    """Parents and lengths of a random binary tree by random splits (the topology of random
    merges): tips get ids 0..tips-1, the root is the last node.  Exponential lengths."""
    rng = np.random.default_rng([int(seed), 1])
    e = tips - 1                                            # split k acts on one of k+1 lineages
    slot = np.floor(rng.random(e) * np.arange(1, e + 1)).astype(np.int64)
    # writes to lineage slots in time order: split k rewrites slot[k] and opens slot k+1
    w_slot = np.stack([slot, np.arange(1, e + 1)], 1).reshape(-1)
    order = np.argsort(w_slot, kind="stable")
    s_slot = w_slot[order]
    prev = np.full(2 * e, -1, dtype=np.int64)
    same = np.flatnonzero(s_slot[1:] == s_slot[:-1]) + 1
    prev[order[same]] = order[same - 1]                     # the write this one replaces
    # write 2k (slot[k]) and write 2k+1 (the opened slot) are split k's two children; the node
    # split by k is the write that split k's first write replaces (-1: the root)
    split = prev[0::2]
    ident = np.full(2 * e, -1, dtype=np.int64)              # node id of each write
    inner = np.flatnonzero(split >= 0)
    ident[split[inner]] = 2 * tips - 2 - inner              # the node that split k divides
    left = np.flatnonzero(ident < 0)
    ident[left] = rng.permutation(left.shape[0])            # never split: tips
    parent = np.full(2 * tips - 1, -1, dtype=np.int64)
    parent[ident] = 2 * tips - 2 - np.arange(2 * e) // 2
    length = rng.exponential(0.05, size=2 * tips - 1)
    length[-1] = 0.0
    return parent, length


def _table(tips, samples, nnz, law, seed, stream=2, depth=0):
    """(indptr, tips, counts), ragged: nnz/2 to 3 nnz/2 distinct tips per sample, by popularity
    (Zipf, exponent 1.1) or uniform; counts round(LogNormal(2, 1.5)) + 1, or with depth > 0
    that many reads per sample."""
    g = _gen(seed, stream)
    most = max(1, min(tips, nnz + nnz // 2))
    size = torch.randint(max(1, nnz // 2), most + 1, (samples,), generator=g, device=DEV)
    logw = torch.zeros(tips, device=DEV)
    if law == "zipf":
        rank = torch.randperm(tips, generator=g, device=DEV).float() + 1.0
        logw = -1.1 * torch.log(rank)
    step = max(1, (1 << 28) // tips)
    picks = []
    for r0 in range(0, samples, step):
        rows = min(step, samples - r0)
        u = torch.rand((rows, tips), generator=g, device=DEV).clamp_(1e-7, 1.0 - 1e-7)
        u.log_().neg_().log_().neg_().add_(logw)            # Gumbel keys: the largest are a draw
        picks.append(torch.topk(u, most, dim=1, sorted=True).indices)
    pick = torch.cat(picks)
    cnt = torch.round(torch.exp(torch.randn((samples, most), generator=g, device=DEV) * 1.5 + 2.0)) + 1.0
    keep = torch.arange(most, device=DEV)[None, :] < size[:, None]
    if depth:
        reads = torch.multinomial(torch.where(keep, cnt, torch.zeros_like(cnt)), depth,
                                  replacement=True, generator=g)
        cnt = torch.zeros_like(cnt).scatter_add_(1, reads, torch.ones_like(reads, dtype=cnt.dtype))
        keep = cnt > 0
    indptr = np.zeros(samples + 1, dtype=np.int64)
    np.cumsum(keep.sum(1).cpu().numpy(), out=indptr[1:])
    return indptr, pick[keep].cpu().numpy(), cnt[keep].long().cpu().numpy()


def _points(samples, dim, seed, stream):
    """Points with a falling spectrum; their distances stand for a study's matrix."""
    g = _gen(seed, stream)
    scale = 0.85 ** torch.arange(dim, device=DEV, dtype=torch.float64)
    return torch.randn((samples, dim), generator=g, device=DEV, dtype=torch.float64) * scale


def _condensed(square):
    n = square.shape[0]
    i, j = torch.triu_indices(n, n, 1, device=DEV)
    return square[i, j].contiguous()


def _distances(points):
    sq = (points * points).sum(1)
    d2 = sq[:, None] + sq[None, :] - 2.0 * points @ points.T
    d = d2.clamp_min_(0.0).sqrt_()
    return d / d.max()


def _weights(dims, seed):
    rng = np.random.default_rng([int(seed), 7])
    out = []
    for a, b in zip(dims[:-1], dims[1:]):
        lim = math.sqrt(6.0 / a)
        out.append((rng.uniform(-lim, lim, size=(b, a)).astype(np.float32),
                    rng.normal(0.0, 0.01, size=b).astype(np.float32)))
    skip = (rng.standard_normal((dims[-1], dims[0])) / math.sqrt(dims[0])).astype(np.float32)
    return out, skip


def _dims(case):
    return [case["d0"], case["hidden"], case["hidden"], case["dz"]]


def _projection(nodes, d0, seed):
    """Four distinct output dimensions per node, each with a sign."""
    rng = np.random.default_rng([int(seed), 6])
    first = rng.integers(0, d0, size=nodes)
    dims = (first[:, None] + np.arange(4)[None, :] * (d0 // 4)
            + rng.integers(0, d0 // 4, size=(nodes, 4))) % d0
    while True:
        srt = np.sort(dims, axis=1)
        dup = np.any(srt[:, 1:] == srt[:, :-1], axis=1)
        if not dup.any():
            break
        dims[dup] = rng.integers(0, d0, size=(int(dup.sum()), 4))
    signs = np.where(rng.random((nodes, 4)) < 0.5, -1, 1)
    return dims.astype(np.int32), signs.astype(np.int8)


def _z_of(table, tips, dz, seed):
    """A linear map of a table's proportions to dz dimensions (what the encoder yields: samples
    that share abundant tips lie near each other)."""
    indptr, tp, ct = table
    g = _gen(seed, 21)
    basis = torch.randn((tips, dz), generator=g, device=DEV)
    n = indptr.shape[0] - 1
    sizes = np.diff(indptr)
    most = int(sizes.max())
    pad_t = np.zeros((n, most), dtype=np.int64)
    pad_w = np.zeros((n, most), dtype=np.float32)
    mask = np.arange(most)[None, :] < sizes[:, None]
    pad_t[mask], pad_w[mask] = tp, ct
    pad_w = np.sqrt(pad_w / pad_w.sum(1, keepdims=True))
    out = torch.empty((n, dz), device=DEV)
    for r0 in range(0, n, 512):
        t = torch.as_tensor(pad_t[r0:r0 + 512], device=DEV)
        w = torch.as_tensor(pad_w[r0:r0 + 512], device=DEV)
        out[r0:r0 + 512] = (basis[t] * w[..., None]).sum(1)
    return out


def _batch_tables(case, seed):
    lo, hi, nnz = case["n_min"], case["n_max"], min(case["nnz"], case["tips"] // 2)
    sizes = [lo + int((hi - lo) * ((r + 1) * 0.6180339887 % 1.0)) for r in range(case["tables"])]
    return [_table(case["tips"], n, nnz, "zipf", seed, stream=30 + r, depth=case["depth"])
            for r, n in enumerate(sizes)]


def _out(case):
    return torch.float64 if case["out"] == "f64" else torch.float32


def _stripes(case):
    s = case["samples"] // 2
    p = case["pieces"]
    return s * (p // 2) // p, s * (p // 2 + 1) // p


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind in ("dm", "step", "encode"):
        parent, length = _tree(case["tips"], seed)
        s["tree"] = uf.Tree(parent, length)
        nnz = min(case["nnz"], case["tips"] // 2)
        table = uf.Table(s["tree"], *_table(case["tips"], case["samples"], nnz,
                                            case.get("law", "zipf"), seed))
        s["emb"] = uf.Embedding(s["tree"], table)
    if kind == "encode":
        s["dims"], s["signs"] = _projection(2 * case["tips"] - 1, case["d0"], seed)
        params, skip = _weights(_dims(case), seed)
        s["mlp"] = uf.MLP(_dims(case), max_rows=max(case["samples"], 2), params=params, skip=skip)
    elif kind == "batch":
        parent, length = _tree(case["tips"], seed)
        s["tree"] = uf.Tree(parent, length)
        s["batch"] = uf.Batch(s["tree"], [uf.Table(s["tree"], *t) for t in _batch_tables(case, seed)])
        if case["precision"] != "fp32":
            s["batch"].set_precision(case["precision"])
    elif kind == "pcoa":
        d = _distances(_points(case["samples"], 40, seed, 11))
        s["dm"] = _condensed(d)
        a = -0.5 * d * d
        s["rm"] = a.mean(1) if case["means"] else None
        s["gm"] = a.mean(1).mean().reshape(1) if case["means"] else None
        s["omega"] = torch.randn((case["samples"], case["cols"]), generator=_gen(seed, 12), device=DEV,
                                 dtype=torch.float64)
    elif kind == "mantel":
        s["x"], s["y"], s["perms"] = _mantel_inputs(case, seed)
    elif kind == "train":
        params, skip = _weights(_dims(case), seed)
        s["mlp"] = uf.MLP(_dims(case), max_rows=3 * case["triples"], params=params, skip=skip)
        s.update(_triples(case, seed))
        s["step"] = 0
    elif kind == "place":
        parent, length = _tree(case["tips"], seed)
        s["tree"] = uf.Tree(parent, length)
        for name, n, stream in (("r", case["refs"], 2), ("q", case["queries"], 3)):
            t = _place_table(case, seed, n, stream)
            s["z_" + name] = _z_of(t, case["tips"], case["dz"], seed)
            s["s_" + name] = uf.Sparse(uf.Embedding(s["tree"], uf.Table(s["tree"], *t)))
    return s


def _place_table(case, seed, n, stream):
    return _table(case["tips"], n, min(case["nnz"], case["tips"] // 2), "zipf", seed, stream=stream)


def _mantel_inputs(case, seed):
    n = case["samples"]
    p = _points(n, 30, seed, 13)
    x = _condensed(_distances(p))
    y = _condensed(_distances(p + 0.8 * _points(n, 30, seed, 14)))
    if case["method"] == "spearman":                 # distances come with ties
        y = torch.round(y * 4096.0) / 4096.0
    keys = torch.rand((case["perms"], n), generator=_gen(seed, 15), device=DEV)
    return x, y, torch.argsort(keys, dim=1).to(torch.int32)


def _triples(case, seed):
    g = _gen(seed, 16)
    x = (torch.randn((case["rows"], case["d0"]), generator=g, device=DEV) * 0.05).to(torch.bfloat16)
    shape = (case["steps"], case["triples"])
    idx = torch.randint(0, case["rows"], (3,) + shape, generator=g, device=DEV, dtype=torch.int32)
    near = torch.rand(shape, generator=g, device=DEV) * 0.4 + 0.2
    far = near + torch.rand(shape, generator=g, device=DEV) * 0.3
    return {"x": x, "idx": idx, "near": near, "far": far}


LR, TAU, ALPHA = 1e-4, 0.03, 0.1      # training step
SCALE = 8.0                           # of the projection's outputs


# --------------------------------------------------------------------------- one pass
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "dm":
        if case["pieces"] > 1:
            b, e = _stripes(case)
            d, sums = uf.dm_stripes(s["emb"], case["variant"], case["precision"], b, e,
                                    out_dtype=_out(case), row_sums=case["means"])
            return [d, sums]
        return list(uf.dm(s["emb"], case["variant"], case["precision"], out_dtype=_out(case),
                          row_means=case["means"]))
    if kind == "step":
        s["emb"].prepare(scalars=True, split_weighted=True, split_unweighted=True)
        return [list(uf.dm(s["emb"], "weighted", "fp32_split", row_means=True)),
                list(uf.dm(s["emb"], "unweighted", "mfma_split", row_means=True))]
    if kind == "batch":
        return s["batch"].run()
    if kind == "pcoa":
        return list(uf.pcoa(s["dm"], case["samples"], case["dims"], s["omega"],
                            power_iters=case["iters"], row_means=s["rm"], grand_mean=s["gm"]))
    if kind == "mantel":
        return list(uf.mantel(s["x"], s["y"], case["samples"], case["method"], s["perms"],
                              alternative=case["alternative"]))
    if kind == "train":
        m = s["mlp"]
        losses = []
        for k in range(case["steps"]):
            s["step"] += 1
            losses.append(m.triplet_loss_grad(s["x"], s["idx"][0, k], s["idx"][1, k], s["idx"][2, k],
                                              s["near"][k], s["far"][k], tau=TAU, dist_weight=ALPHA))
            m.adam(LR, s["step"])
        return losses + [list(m.get(k)) for k in range(m.n_layers + 1)]
    if kind == "encode":
        x = uf.project(s["tree"], s["emb"], s["dims"], s["signs"], out_dim=case["d0"], scale=SCALE)
        return [x, s["mlp"].forward(x)]
    return list(placement.place(s["z_r"], s["z_q"], s["s_q"], s["s_r"], case["candidates"], case["k"]))


# --------------------------------------------------------------------------- work
def _touched(tips, nnz):
    """Branches a sample of nnz tips touches on a random tree of that many tips."""
    nnz = max(1, min(nnz, tips // 2))
    return min(2 * tips - 2, nnz * (2.0 * math.log(tips / nnz) + 1.0))


def work(case):
    kind = case["kind"]
    if kind in ("dm", "step"):
        n, nnz = case["samples"], min(case["nnz"], case["tips"] // 2)
        pairs = n * (n - 1) / 2
        table = n * nnz * 12 + case["tips"] * 2 * 16
        if kind == "step":
            return {"bytes": table + 2 * 8 * pairs, "flops": 4 * pairs * _touched(case["tips"], nnz)}
        pairs /= case["pieces"]
        return {"bytes": table + pairs * (8 if case["out"] == "f64" else 4),
                "flops": 2 * pairs * _touched(case["tips"], nnz)}
    if kind == "batch":
        n = (case["n_min"] + case["n_max"]) / 2
        nnz = min(case["nnz"], case["tips"] // 2)
        pairs = case["tables"] * n * n / 2
        return {"bytes": case["tables"] * n * nnz * 12 + 4 * pairs,
                "flops": 2 * pairs * _touched(case["tips"], nnz)}
    if kind == "pcoa":
        n = case["samples"]
        return {"bytes": 4.0 * n * n + 8 * n * (case["cols"] + case["dims"]),
                "flops": 2.0 * n * n * case["cols"] * (case["iters"] + 2)}
    if kind == "mantel":
        n = case["samples"]
        return {"bytes": 8.0 * n * n + 4.0 * n * case["perms"], "flops": 1.0 * n * n * case["perms"]}
    if kind in ("train", "encode"):
        d = _dims(case)
        rows = 3 * case["triples"] if kind == "train" else case["samples"]
        mac = sum(a * b for a, b in zip(d[:-1], d[1:])) + d[0] * d[-1]
        if kind == "train":
            grad = d[1] * d[2] + d[2] * d[3]
            return {"bytes": case["steps"] * (26.0 * mac + 2 * rows * d[0]),
                    "flops": 2.0 * case["steps"] * rows * (2 * mac + grad)}
        nnz = min(case["nnz"], case["tips"] // 2)
        return {"bytes": rows * (nnz * 12 + 2 * d[0] + 4 * d[-1]) + 2 * mac + case["tips"] * 2 * 36,
                "flops": 2.0 * rows * (mac + 4 * _touched(case["tips"], nnz))}
    nq, nr = case["queries"], case["refs"]
    t = _touched(case["tips"], case["nnz"])
    return {"bytes": 4.0 * (nq + nr) * case["dz"] + 12.0 * (nq + min(nr, nq * case["candidates"])) * t
            + nq * (4 * case["candidates"] + 12 * case["k"]),
            "flops": 3.0 * nq * nr * case["dz"] + 2.0 * nq * case["candidates"] * t}


# --------------------------------------------------------------------------- in 64 bits
def _dense(parent, table, tips):
    """Counts under every non-root node, [nodes - 1][samples] in 64 bits."""
    indptr, tp, ct = table
    n = indptr.shape[0] - 1
    c = torch.zeros((2 * tips - 1, n), dtype=torch.float64, device=DEV)
    rows = torch.as_tensor(np.repeat(np.arange(n), np.diff(indptr)), device=DEV)
    c[torch.as_tensor(tp, device=DEV), rows] = torch.as_tensor(ct, device=DEV).double()
    depth = np.zeros(2 * tips - 1, dtype=np.int64)
    for v in range(2 * tips - 3, -1, -1):            # a parent's id exceeds its children's
        depth[v] = depth[parent[v]] + 1
    order = np.argsort(-depth, kind="stable")
    cuts = np.flatnonzero(np.diff(depth[order])) + 1
    for nodes in np.split(order, cuts):
        nodes = nodes[parent[nodes] >= 0]
        if nodes.size:
            c.index_add_(0, torch.as_tensor(parent[nodes], device=DEV),
                         c[torch.as_tensor(nodes, device=DEV)])
    return c[:-1]


def _weighted(c, length):
    x = (c / c_total(c, length)[None, :]) * length[:, None]
    num = torch.cdist(x.T.contiguous(), x.T.contiguous(), p=1)
    den = x.sum(0)
    den = den[:, None] + den[None, :]
    return torch.where(den > 0, num / den, torch.zeros_like(num))


def c_total(c, length):
    """Sample totals: the tips are the first rows."""
    return c[: (length.shape[0] + 2) // 2].sum(0)


def _unweighted(c, length):
    a = (c > 0).double()
    gram = (a * length[:, None]).T @ a
    w = torch.diagonal(gram)
    both = w[:, None] + w[None, :] - gram
    return torch.where(both > 0, (both - gram) / both, torch.zeros_like(both))


def _as_stripes(square, b, e):
    n = square.shape[0]
    i = torch.arange(n, device=DEV)[None, :]
    j = (i + torch.arange(b, e, device=DEV)[:, None] + 1) % n
    return square[i.expand_as(j), j]


def _exact_dm(square, means):
    a = -0.5 * square * square
    a.fill_diagonal_(0.0)
    rm = a.mean(1)
    return [_condensed(square), rm if means else None, rm.mean().reshape(1) if means else None]


def exact(case, seed):
    kind = case["kind"]
    n = case.get("samples", 0)
    if kind in ("dm", "step", "batch", "encode", "place"):
        parent, length = _tree(case["tips"], seed)
        lt = torch.as_tensor(length[:-1], device=DEV)
    if kind in ("dm", "step"):
        table = _table(case["tips"], n, min(case["nnz"], case["tips"] // 2), case["law"], seed)
        c = _dense(parent, table, case["tips"])
        slow = n * n * 2.0 * case["tips"] > 1.5e12      # sums of |x - y| over every pair
        if kind == "step":
            return [_exact_dm(_weighted(c, lt), True) if not slow else [None, None, None],
                    _exact_dm(_unweighted(c, lt), True)]
        if case["variant"] == "weighted":
            if slow:
                return None
            square = _weighted(c, lt)
        else:
            square = _unweighted(c, lt)
        if case["pieces"] > 1:
            b, e = _stripes(case)
            sums = None
            if case["means"]:
                q = -0.5 * _as_stripes(square, b, e) ** 2
                i = torch.arange(n, device=DEV)[None, :].expand_as(q)
                j = (i + torch.arange(b, e, device=DEV)[:, None] + 1) % n
                if n % 2 == 0 and e == n // 2 and e > b:
                    q[-1, n // 2:] = 0.0                 # the last stripe holds its pairs twice
                sums = torch.zeros(n, dtype=torch.float64, device=DEV)
                sums.index_add_(0, i.reshape(-1), q.reshape(-1))
                sums.index_add_(0, j.reshape(-1), q.reshape(-1))
            return [_as_stripes(square, b, e), sums]
        return _exact_dm(square, case["means"])
    if kind == "batch":
        return [_condensed(_weighted(_dense(parent, t, case["tips"]), lt))
                for t in _batch_tables(case, seed)]
    if kind == "pcoa":
        return _exact_pcoa(case, seed)
    if kind == "mantel":
        return _exact_mantel(case, seed)
    if kind == "train":
        return _exact_train(case, seed)
    if kind == "encode":
        table = _table(case["tips"], n, min(case["nnz"], case["tips"] // 2), "zipf", seed)
        c = _dense(parent, table, case["tips"])
        y = (c / c_total(c, lt)[None, :]) * lt[:, None] * (0.5 * SCALE)
        dims, signs = _projection(2 * case["tips"] - 1, case["d0"], seed)
        x = torch.zeros((case["d0"], n), dtype=torch.float64, device=DEV)
        for j in range(4):
            x.index_add_(0, torch.as_tensor(dims[:-1, j], device=DEV).long(),
                         y * torch.as_tensor(signs[:-1, j], device=DEV).double()[:, None])
        params, skip = _weights(_dims(case), seed)
        return [x.T.contiguous(), _forward(x.T.contiguous(), *_params64(params, skip))]
    return _exact_place(case, seed, parent, lt)


def _exact_pcoa(case, seed):
    n = case["samples"]
    d = _distances(_points(n, 40, seed, 11))
    d.fill_diagonal_(0.0)
    a = -0.5 * d * d
    a = 0.5 * (a + a.T)
    r, g = a.mean(1), a.mean()
    b = a - r[:, None] - r[None, :] + g
    q, _ = torch.linalg.qr(b @ torch.randn((n, case["cols"]), generator=_gen(seed, 12), device=DEV,
                                           dtype=torch.float64))
    for _ in range(case["iters"]):
        q, _ = torch.linalg.qr(b @ q)
    lam, w = np.linalg.eigh((q.T @ (b @ q)).cpu().numpy())
    lam, w = lam[::-1][: case["dims"]].copy(), w[:, ::-1][:, : case["dims"]].copy()
    coords = q @ torch.as_tensor(w * np.sqrt(np.maximum(lam, 0.0)), device=DEV)
    top = coords.abs().argmax(0)
    sign = torch.sign(coords[top, torch.arange(case["dims"], device=DEV)])
    return [coords * sign, lam, float(-n * g)]


def _ranks(v):
    u, inv, cnt = torch.unique(v, return_inverse=True, return_counts=True)
    last = torch.cumsum(cnt, 0).double()
    return (last - 0.5 * (cnt.double() - 1.0))[inv]


def _exact_mantel(case, seed):
    n = case["samples"]
    x, y, perms = _mantel_inputs(case, seed)
    if case["method"] == "spearman":
        x, y = _ranks(x), _ranks(y)
    x = x - x.mean()
    y = y - y.mean()
    x, y = x / x.norm(), y / y.norm()
    i, j = torch.triu_indices(n, n, 1, device=DEV)
    full = torch.zeros((n, n), dtype=torch.float64, device=DEV)
    full[i, j] = x
    full = full + full.T
    ysq = torch.zeros((n, n), dtype=torch.float64, device=DEV)
    ysq[i, j] = y
    stat = float((x * y).sum())
    ps = np.array([float((full[p][:, p] * ysq).sum()) for p in perms.long()])
    more = {"two-sided": np.abs(ps) >= abs(stat), "greater": ps >= stat, "less": ps <= stat}
    return [stat, float(more[case["alternative"]].sum() + 1) / (case["perms"] + 1), ps]


def _params64(params, skip):
    return ([(torch.as_tensor(w, device=DEV).double(), torch.as_tensor(b, device=DEV).double())
             for w, b in params], torch.as_tensor(skip, device=DEV).double())


def _forward(x, params, skip):
    h = x
    for k, (w, b) in enumerate(params):
        h = h @ w.T + b
        if k + 1 < len(params):
            h = torch.relu(h)
    return h + x @ skip.T


def _exact_train(case, seed):
    params, skip = _params64(*_weights(_dims(case), seed))
    t = _triples(case, seed)
    leaf = [v.requires_grad_(True) for pair in params for v in pair] + [skip.requires_grad_(True)]
    m = [torch.zeros_like(v) for v in leaf]
    u = [torch.zeros_like(v) for v in leaf]
    losses = []
    for k in range(case["steps"]):
        z = [_forward(t["x"][t["idx"][e, k].long()].double(), params, skip) for e in range(3)]
        ep, en = (z[0] - z[1]).norm(dim=1), (z[0] - z[2]).norm(dim=1)
        loss = (ALPHA * ((ep - t["near"][k].double()) ** 2 + (en - t["far"][k].double()) ** 2)
                + TAU * torch.nn.functional.softplus((ep - en) / TAU, threshold=1e9)).mean()
        grads = torch.autograd.grad(loss, leaf)
        losses.append(loss.detach().reshape(1))
        with torch.no_grad():
            for v, gr, a, b in zip(leaf, grads, m, u):
                a.mul_(0.9).add_(gr, alpha=0.1)
                b.mul_(0.999).add_(gr * gr, alpha=0.001)
                v -= LR * (a / (1 - 0.9 ** (k + 1))) / ((b / (1 - 0.999 ** (k + 1))).sqrt() + 1e-8)
    out = [v.detach() for v in leaf]
    return losses + [[out[2 * k], out[2 * k + 1]] for k in range(len(params))] + [[out[-1], None]]


def _exact_place(case, seed, parent, lt):
    parts = {}
    for name, n, stream in (("r", case["refs"], 2), ("q", case["queries"], 3)):
        table = _place_table(case, seed, n, stream)
        z = _z_of(table, case["tips"], case["dz"], seed).double()
        c = _dense(parent, table, case["tips"])
        parts[name] = (z, ((c / c_total(c, lt)[None, :]) * lt[:, None]).T.contiguous())
    (zr, xr), (zq, xq) = parts["r"], parts["q"]
    near = torch.cdist(zq, zr, compute_mode="donot_use_mm_for_euclid_dist")
    cand = torch.topk(near, case["candidates"], dim=1, largest=False).indices
    best = torch.empty((case["queries"], case["k"]), dtype=torch.float64, device=DEV)
    sr = xr.sum(1)
    for i in range(case["queries"]):
        x = xr[cand[i]]
        d = (x - xq[i][None, :]).abs().sum(1) / (sr[cand[i]] + xq[i].sum())
        best[i] = torch.topk(d, case["k"], largest=False, sorted=True).values
    return [None, best, None]

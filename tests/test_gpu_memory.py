"""Workspace of large unweighted matrices and of batches of very many tables: bounded by the
results and the chunk, and the parts that they are then taken in give the same bits."""
import numpy as np
import pytest

import paper_2107_05397_amd as uf
import synth

from ._util import random_rows, table as make_table

pytestmark = pytest.mark.gpu

GIB = 1 << 30


def _embedding(n, n_tips, seed):
    import torch  # noqa: F401
    rng = np.random.default_rng(seed)
    tree = synth.gen_tree(n_tips, 0.05, seed)
    some = random_rows(rng, np.arange(n_tips), 500, max_nnz=n_tips // 6)
    table = make_table([some[k] for k in rng.integers(0, 500, n)])
    t = uf.Tree(tree.parent, tree.length)
    return uf.Embedding(t, uf.Table(t, table.indptr, table.tips, table.counts))


def test_unweighted_workspace_holds_one_sum_per_pair():
    n = 60000
    emb = _embedding(n, 60, 1)
    for precision, elem in (("fp64", 8), ("fp32", 4), ("mfma", 4)):
        for means in (False, True):
            got = uf.workspace_size(emb, "unweighted", precision, row_stats=means)
            assert got <= (elem + 8 * means) * (n // 2) * n + (9 + 2 * means) * GIB, (precision, means)
    few = uf.workspace_size(_embedding(300, 60, 2), "unweighted", "fp64")
    assert few <= 64 << 20


# just above 16 GiB of sums: two parts; even and odd
@pytest.mark.parametrize("n,precision", [(46400, "fp64"), (46501, "fp64"), (65700, "fp32")])
def test_unweighted_in_parts(n, precision):
    import torch
    emb = _embedding(n, 60, n)
    dtype = torch.float64 if precision == "fp64" else torch.float32
    full, rm, gm = uf.dm(emb, "unweighted", precision, out_dtype=dtype, row_means=True)
    s = n // 2
    buf = torch.full_like(full, -1.0)
    for k in range(4):
        uf.dm_stripes(emb, "unweighted", precision, s * k // 4, s * (k + 1) // 4, layout="condensed", out=buf)
    assert torch.equal(buf, full)
    del buf
    stripes, _ = uf.dm_stripes(emb, "unweighted", precision, 0, s, out_dtype=dtype)
    g = torch.Generator(device="cuda").manual_seed(n)
    a = torch.randint(0, s, (1 << 20,), generator=g, device="cuda")
    i = torch.randint(0, n, (1 << 20,), generator=g, device="cuda")
    j = (i + a + 1) % n
    lo, hi = torch.minimum(i, j), torch.maximum(i, j)
    assert torch.equal(stripes[a, i], full[lo * n - lo * (lo + 1) // 2 + hi - lo - 1])
    # row means of -d^2/2 from the stripes: n terms of at most 1/2, each rounded, in any order
    # (from FP32 distances: each of d <= 1 rounded to 2^-25)
    sums = torch.zeros(n, dtype=torch.float64, device="cuda")
    for t in range(s):
        q = -0.5 * stripes[t].double() ** 2
        if n % 2 == 0 and t == s - 1:
            q[s:] = 0.0
        sums += q + torch.roll(q, t + 1)
    tol = 2.0 ** -53 * (n + 4) + (0.0 if dtype == torch.float64 else 2.0 ** -25)
    assert torch.max(torch.abs(sums / n - rm)).item() <= tol
    assert abs(float(gm) - float(rm.mean())) <= 2.0 ** -53 * (n + 4)


def _tables(tree, sizes, n_tips, seed):
    rng = np.random.default_rng(seed)
    out = []
    for n in sizes:
        x = make_table(random_rows(rng, np.arange(n_tips), n, max_nnz=60))
        out.append(uf.Table(tree, x.indptr, x.tips, x.counts))
    return out


# (sizes, times, tips): tables of few samples, whose blocks of 64 are mostly padding: the
# chunk is sized for these; tables whose segments side by side would take more than 4 GiB:
# one plane each (2,049 tips: 16 segments)
@pytest.mark.parametrize("sizes,times,n_tips", [((2, 3, 5), 1000, 20000), ((576, 575, 300), 190, 2049)])
def test_batches_of_very_many_tables(sizes, times, n_tips):
    import torch
    tree = synth.gen_tree(n_tips, 0.05, n_tips)
    t = uf.Tree(tree.parent, tree.length)
    tabs = _tables(t, sizes, n_tips, n_tips)
    few = uf.Batch(t, tabs)
    want = [o.clone() for o in few.run()]
    for tb, w in zip(tabs, want):
        d, _, _ = uf.dm(uf.Embedding(t, tb), "weighted_normalized", "fp32", out_dtype=torch.float32)
        assert torch.equal(d, w)
    pairs = sum(n // 2 * n for n in sizes) * times
    try:
        for nodes in (0, 900):
            uf.set_chunk_nodes(nodes)
            b = uf.Batch(t, tabs * times)
            uf.set_chunk_nodes(0)
            if nodes == 0:
                chunk = sum((n + 63) // 64 for n in sizes) * times * (tree.n_nodes + 1) * (64 * 4 + 8)
                assert b.workspace_size() <= min(chunk, 17 * GIB) + 2 * 4 * pairs + (64 << 20)
            got = b.run()
            torch.cuda.synchronize()
            for k, g in enumerate(got):
                assert torch.equal(g, want[k % len(sizes)]), (nodes, k)
            for cfg in ((8, 1, 64), (16, 2, 256)):
                b.set_config(*cfg)
                got = b.run()
                torch.cuda.synchronize()
                assert all(torch.equal(g, want[k % len(sizes)]) for k, g in enumerate(got)), cfg
            if nodes == 0:
                assert b.autotune() > 0
            b.close()
            del b, got
            torch.cuda.empty_cache()
    finally:
        uf.set_chunk_nodes(0)

"""Large FP32 weighted matrices of tables that touch many branches run on LDS tiles over all
branches: the bits of the pair tiles (which stripe ranges too small for LDS tiles take), whole,
in chunks, in a batch and as the dense part of a split; and the FP64 oracle."""
import dataclasses

import numpy as np
import pytest

import oracle
import paper_2107_05397_amd as uf
import synth

from ._util import random_rows, table as make_table

pytestmark = pytest.mark.gpu

TIPS = 60


def _inputs(n, seed, lonely=False):
    rng = np.random.default_rng(seed)
    tree = synth.gen_tree(TIPS, 0.05, seed)
    some = random_rows(rng, np.arange(1, TIPS), 700, max_nnz=40)
    rows = [some[k] for k in rng.integers(0, 700, n)]
    rows[-1] = dict(rows[0])
    if lonely:                                                 # a sample of hardly any length
        path, v = [], 0
        while tree.parent[v] >= 0:
            path.append(v)
            v = int(tree.parent[v])
        length = tree.length.copy()
        length[path] = 1e-7
        tree = dataclasses.replace(tree, length=length)
        rows[3] = {0: 5}
    table = make_table(rows)
    t = uf.Tree(tree.parent, tree.length)
    return tree, table, t, uf.Table(t, table.indptr, table.tips, table.counts)


def _pieces(emb, precision, n, like):
    import torch
    buf = torch.full_like(like, -1.0)
    s = n // 2
    for k in range(5):
        uf.dm_stripes(emb, "weighted", precision, s * k // 5, s * (k + 1) // 5, layout="condensed", out=buf)
    return buf


@pytest.mark.parametrize("n", [12400, 12401])
def test_lds_tiles_equal_pair_tiles(n):
    import torch
    tree, table, t, tb = _inputs(n, n)
    emb = uf.Embedding(t, tb)
    full, _, _ = uf.dm(emb, "weighted", "fp32")
    assert torch.equal(_pieces(emb, "fp32", n, full), full)
    assert float(full[n - 2]) == 0.0                           # pair (0, n-1)
    try:
        uf.set_chunk_nodes(50)
        d, _, _ = uf.dm(emb, "weighted", "fp32")
        assert torch.equal(d, full)
    finally:
        uf.set_chunk_nodes(0)
    pick = np.r_[0:100, n - 100:n]
    part = make_table([dict(zip(table.tips[a:b].tolist(), table.counts[a:b].tolist()))
                       for a, b in zip(table.indptr[pick], table.indptr[pick + 1])])
    want = oracle.dm(tree, part, "weighted_normalized")
    i, j = np.triu_indices(len(pick), 1)
    at = pick[i] * n - pick[i] * (pick[i] + 1) // 2 + pick[j] - pick[i] - 1
    # K terms of two rounded values each, over a denominator that bounds the sum of the values
    assert np.max(np.abs(full.cpu().numpy()[at] - want)) <= (tree.n_nodes + 2) * 2.0 ** -24


def test_batch_on_lds_tiles_equals_single_calls():
    import torch
    _, _, t, tb = _inputs(12400, 7)
    rng = np.random.default_rng(8)
    tabs = [tb]
    for n in (4100, 65, 4351):
        x = make_table(random_rows(rng, np.arange(TIPS), n, max_nnz=40))
        tabs.append(uf.Table(t, x.indptr, x.tips, x.counts))
    want = [uf.dm(uf.Embedding(t, x), "weighted", "fp32", out_dtype=torch.float32)[0] for x in tabs]
    try:
        for nodes in (0, 50):
            uf.set_chunk_nodes(nodes)
            b = uf.Batch(t, tabs)
            for g, w in zip(b.run(), want):
                assert torch.equal(g, w), nodes
    finally:
        uf.set_chunk_nodes(0)


def test_split_without_fixed_point():
    import torch
    n = 12400
    _, _, t, tb = _inputs(n, 9, lonely=True)
    try:
        uf.set_split_threshold(0.0, "weighted")                # every touched branch is dense
        emb = uf.Embedding(t, tb)
        full, _, _ = uf.dm(emb, "weighted", "fp32_split")
        assert torch.equal(_pieces(emb, "fp32_split", n, full), full)
        plain, _, _ = uf.dm(emb, "weighted", "fp32")
        assert torch.equal(full, plain)                        # (all branches, in FP32: no fixed point)
    finally:
        uf.set_split_threshold(None, "weighted")

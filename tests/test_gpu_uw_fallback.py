"""Unweighted matrices whose lengths span too wide a range for the digits of the product on
presence bits: pair tiles over touched branches (FP64, FP32) and the BF16 product over all
branches, at the edges of their blocks, segments and chunks, against the FP64 oracle."""
import dataclasses

import numpy as np
import pytest

import oracle
import paper_2107_05397_amd as uf
import synth

from ._util import random_rows, table as make_table

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_tips", [(2, 3), (63, 130), (65, 700), (129, 257), (300, 2600), (1800, 40)])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "mfma"])
def test_sums_of_the_lengths_themselves(n, n_tips, precision):
    import torch
    rng = np.random.default_rng(n)
    tree = synth.gen_tree(n_tips, 0.05, n + n_tips)
    length = tree.length.astype(np.float32).astype(np.float64)
    length[0] = 1e15                                           # tip 0, which no sample holds
    tree = dataclasses.replace(tree, length=length)
    rows = random_rows(rng, np.arange(1, n_tips), n, max_nnz=max(2, n_tips // 6))
    rows[-1] = dict(rows[0])
    table = make_table(rows)
    work = tree
    if precision == "mfma":
        l = torch.tensor(length, dtype=torch.float32)
        hi = l.to(torch.bfloat16).float()
        work = dataclasses.replace(tree, length=(hi.double() + (l - hi).to(torch.bfloat16).double()).numpy())
    want = oracle.dm(work, table, "unweighted")
    t = uf.Tree(tree.parent, tree.length)
    emb = uf.Embedding(t, uf.Table(t, table.indptr, table.tips, table.counts))
    full, _, _ = uf.dm(emb, "unweighted", precision)
    # sums of at most K lengths, each rounded once, in both parts of a quotient of at most 1
    tol = 6 * tree.n_nodes * (2.0 ** -53 if precision == "fp64" else 2.0 ** -24)
    assert np.max(np.abs(full.cpu().numpy() - want)) <= tol
    try:
        for nodes in (40, 256, 512, 700):
            uf.set_chunk_nodes(nodes)
            d, _, _ = uf.dm(emb, "unweighted", precision)
            if precision == "mfma":                            # (chunks are whole steps of the product)
                assert np.max(np.abs(d.cpu().numpy() - want)) <= tol, nodes
            else:
                assert torch.equal(d, full), nodes
    finally:
        uf.set_chunk_nodes(0)
    buf = torch.zeros_like(full)
    s = n // 2
    for b, e in ((0, s // 3), (s // 3, s - s // 4), (s - s // 4, s)):
        uf.dm_stripes(emb, "unweighted", precision, b, e, layout="condensed", out=buf)
    assert torch.equal(buf, full)

"""Unweighted Gram product on presence bits, at the edges of its blocks, windows, staged
batches and ranges, against the FP64 oracle; every chunking; and the paths taken instead
when the branch lengths span too wide a range for its digits."""
import dataclasses

import numpy as np
import pytest

import oracle
import paper_2107_05397_amd as uf
import synth

from ._util import random_rows, table as make_table

pytestmark = pytest.mark.gpu


def _lengths(length, precision):
    """The lengths a precision works with (inputs are FP32 values)."""
    import torch
    if precision != "mfma":
        return length
    l = torch.tensor(length, dtype=torch.float32)
    hi = l.to(torch.bfloat16).float()
    return (hi.double() + (l - hi).to(torch.bfloat16).double()).numpy()


def _inputs(n, n_tips, seed, longest=None):
    rng = np.random.default_rng(seed)
    tree = synth.gen_tree(n_tips, 0.05, seed)
    length = tree.length.astype(np.float32).astype(np.float64)
    if longest is not None:
        length[0] = longest                                    # tip 0's branch
    tree = dataclasses.replace(tree, length=length)
    rows = random_rows(rng, np.arange(1 if longest is not None and n_tips > 1 else 0, n_tips), n,
                       max_nnz=max(2, n_tips // 6))
    if longest is not None:
        rows[0][0] = 3
    return tree, make_table(rows)


def _embed(tree, table):
    t = uf.Tree(tree.parent, tree.length)
    return uf.Embedding(t, uf.Table(t, table.indptr, table.tips, table.counts))


# samples: one block and its edges, two and five blocks; branches: one word, one window
# (8,192) and more, lists longer than a staged batch (1,024) and one range (256)
@pytest.mark.parametrize("n,n_tips", [(2, 2), (3, 33), (63, 130), (64, 40), (65, 700), (129, 6000),
                                      (300, 600)])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "mfma"])
def test_bits_match_oracle(n, n_tips, precision):
    import torch
    tree, table = _inputs(n, n_tips, 5 * n + n_tips)
    emb = _embed(tree, table)
    work = dataclasses.replace(tree, length=_lengths(tree.length, precision))
    want = oracle.dm(work, table, "unweighted")
    full, _, _ = uf.dm(emb, "unweighted", precision)
    # digits: 56 (FP64) or 28 bits below the longest branch; each pair's sums are off by
    # at most the rounding of all lengths, d by twice that over the smallest w; plus FP64
    # sums of at most K terms
    l = work.length[:-1]
    q = 2.0 ** (np.ceil(np.log2(l.max())) + 1 - (56 if precision == "fp64" else 28))
    _, w = emb.scalars()
    tol = 2 * l.size * (q / 2) / w.min() + 8 * l.size * 2.0 ** -53
    assert np.max(np.abs(full.cpu().numpy() - want)) <= tol
    try:
        for nodes in (40, 256, 700, 9000):
            uf.set_chunk_nodes(nodes)
            d, _, _ = uf.dm(emb, "unweighted", precision)
            assert torch.equal(d, full), nodes
    finally:
        uf.set_chunk_nodes(0)
    buf = torch.zeros_like(full)
    s = n // 2
    for b, e in ((0, s // 3), (s // 3, s - s // 4), (s - s // 4, s)):
        uf.dm_stripes(emb, "unweighted", precision, b, e, layout="condensed", out=buf)
    assert torch.equal(buf, full)


# one branch so long that the others' digits would be lost (28 bits below 1e9 are 4)
@pytest.mark.parametrize("precision,longest,tol", [("fp64", 1e15, 1e-12), ("fp32", 1e9, 1e-4),
                                                   ("mfma", 1e9, 1e-4)])
def test_wide_length_range_matches_oracle(precision, longest, tol):
    tree, table = _inputs(70, 90, 4, longest)
    want = oracle.dm(dataclasses.replace(tree, length=_lengths(tree.length, precision)), table,
                     "unweighted")
    d, _, _ = uf.dm(_embed(tree, table), "unweighted", precision)
    got = d.cpu().numpy()
    # pairs without sample 0 (whose own sums hold the long branch and round at its scale)
    assert np.max(np.abs(got[69:] - want[69:])) <= tol

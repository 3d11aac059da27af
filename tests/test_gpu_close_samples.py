"""Weighted distances of samples that hardly differ: as small as they are, each term |x - y|
keeps its digits (a difference of large sums would not)."""
import numpy as np
import pytest

import oracle
import paper_2107_05397_amd as uf
import synth

from ._util import table as make_table, tree as make_tree

pytestmark = pytest.mark.gpu


# samples: a pair, across two blocks, more blocks (several segments); reads moved: 1 of 2^20
# and of 2^44
@pytest.mark.parametrize("n,n_tips", [(2, 40), (70, 700), (200, 3000)])
@pytest.mark.parametrize("depth", [1 << 20, 1 << 44])
def test_close_samples_keep_relative_accuracy(n, n_tips, depth):
    import torch  # noqa: F401
    rng = np.random.default_rng(n)
    inner = synth.gen_tree(n_tips, 0.05, n_tips)
    root = int(np.flatnonzero(inner.parent == -1)[0])
    m = inner.n_nodes                           # under a new root: that tree and one tip, m
    parent = np.r_[inner.parent, m + 1, -1]
    parent[root] = m + 1
    tree = make_tree(parent, np.r_[inner.length, 0.5, 0.0])
    pick = rng.permutation(n_tips)
    base, free = pick[:n_tips // 3], pick[n_tips // 3:]
    rows = []
    for s in range(n):                          # a read on each base tip, one on a free tip of
        r = {int(t): 1 for t in base}           # its own, the others on tip m
        r[int(free[s % len(free)])] = 1
        r[m] = depth - sum(r.values())
        rows.append(r)
    table = make_table(rows)
    want = oracle.dm(tree, table, "weighted_normalized")
    assert 0 < want.max() < 100.0 / depth       # (equal samples, where tips repeat: 0)
    t = uf.Tree(tree.parent, tree.length)
    emb = uf.Embedding(t, uf.Table(t, table.indptr, table.tips, table.counts))
    d, _, _ = uf.dm(emb, "weighted_normalized", "fp64")
    # the samples differ on branches of at most len(base) + 1 reads, by one: x = l (c / T) has
    # two roundings, so |x - y| is off by 4 c eps of itself; sums of K terms over sums of K
    # terms; and the oracle's own the same again
    rel = 2 * (2 * tree.n_nodes + 8 + 4 * (len(base) + 1)) * 2.0 ** -53
    assert np.all(np.abs(d.cpu().numpy() - want) <= rel * want)

"""Touched-branch pair tiles (FP64, and FP32 unweighted) at the edges of their blocks,
segments and chunks, against the FP64 oracle; equal samples; every chunking."""
import numpy as np
import pytest

import oracle
import paper_2107_05397_amd as uf
import synth

from ._util import random_rows, table as make_table

pytestmark = pytest.mark.gpu


def _inputs(n, n_tips, seed):
    rng = np.random.default_rng(seed)
    tree = synth.gen_tree(n_tips, 0.05, seed)
    rows = random_rows(rng, np.arange(n_tips), n, max_nnz=max(2, n_tips // 6))
    rows[-1] = dict(rows[0])                                   # equal samples: d = 0 exactly
    return tree, make_table(rows)


# (samples, tips): one block, its edges, two and five blocks; one window of branches, a
# window and one branch, several windows and segments
@pytest.mark.parametrize("n,n_tips", [(2, 2), (3, 129), (63, 130), (64, 40), (65, 700), (129, 257),
                                      (300, 600)])
@pytest.mark.parametrize("variant,precision", [("weighted_normalized", "fp64"), ("unweighted", "fp64"),
                                               ("unweighted", "fp32")])
def test_pair_tiles_match_oracle(n, n_tips, variant, precision):
    import torch
    tree, table = _inputs(n, n_tips, 7 * n + n_tips)
    t = uf.Tree(tree.parent, tree.length)
    emb = uf.Embedding(t, uf.Table(t, table.indptr, table.tips, table.counts))
    want = oracle.dm(tree, table, variant)
    full, _, _ = uf.dm(emb, variant, precision)
    # sums of at most K non-negative terms, each rounded once: relative error K eps in each
    # of the (at most four) sums of a quotient of at most 1
    tol = 6 * tree.n_nodes * (2.0 ** -53 if precision == "fp64" else 2.0 ** -24)
    assert np.max(np.abs(full.cpu().numpy() - want)) <= tol
    if n > 2 and variant == "weighted_normalized":
        assert float(full[n - 2]) == 0.0                       # pair (0, n-1)
    # chunks that cut windows and segments, and stripe ranges, give the same bits
    try:
        for nodes in (40, 256, 512, 700):
            uf.set_chunk_nodes(nodes)
            d, _, _ = uf.dm(emb, variant, precision)
            assert torch.equal(d, full), nodes
    finally:
        uf.set_chunk_nodes(0)
    buf = torch.zeros_like(full)
    s = n // 2
    for b, e in ((0, s // 3), (s // 3, s - s // 4), (s - s // 4, s)):
        uf.dm_stripes(emb, variant, precision, b, e, layout="condensed", out=buf)
    assert torch.equal(buf, full)

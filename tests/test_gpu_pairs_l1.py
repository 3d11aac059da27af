"""FP32 weighted pair tiles (sums of |x - y| over the branches either side touches) at the
edges of their blocks, segments, chunks and tile widths, against the FP64 oracle; the
batch launch of the same tiles against single calls, bit for bit."""
import numpy as np
import pytest

import oracle
import paper_2107_05397_amd as uf
import synth

from ._util import random_rows, table as make_table

pytestmark = pytest.mark.gpu


def _table(n, n_tips, seed):
    rng = np.random.default_rng(seed)
    rows = random_rows(rng, np.arange(n_tips), n, max_nnz=max(2, n_tips // 6))
    rows[-1] = dict(rows[0])                                   # equal samples: d = 0 exactly
    return make_table(rows)


# one block, its edges, several; one window of branches, a window and one branch, several
# segments; 4,095 and 4,096 samples: the last with 8 and the first with 16 samples i a wave
@pytest.mark.parametrize("n,n_tips", [(2, 2), (3, 129), (63, 130), (64, 40), (65, 700), (129, 257),
                                      (300, 600), (4095, 60), (4096, 60)])
def test_l1_tiles_match_oracle(n, n_tips):
    import torch
    tree, table = synth.gen_tree(n_tips, 0.05, n + n_tips), _table(n, n_tips, 5 * n + n_tips)
    t = uf.Tree(tree.parent, tree.length)
    emb = uf.Embedding(t, uf.Table(t, table.indptr, table.tips, table.counts))
    # the oracle on all samples, or on the first and last of a large matrix
    pick = np.arange(n) if n < 1000 else np.r_[0:150, n - 150:n]
    rows = [slice(table.indptr[i], table.indptr[i + 1]) for i in pick]
    part = make_table([dict(zip(table.tips[r].tolist(), table.counts[r].tolist())) for r in rows])
    want = oracle.dm(tree, part, "weighted_normalized")
    a, b = np.triu_indices(len(pick), 1)
    at = pick[a] * n - pick[a] * (pick[a] + 1) // 2 + pick[b] - pick[a] - 1
    full, _, _ = uf.dm(emb, "weighted_normalized", "fp32")
    # at most K terms, each of two rounded values and added with one rounding, over a
    # denominator that bounds the sum of the values
    assert np.max(np.abs(full.cpu().numpy()[at] - want)) <= (tree.n_nodes + 2) * 2.0 ** -24
    if n > 2:
        assert float(full[n - 2]) == 0.0                       # pair (0, n-1)
    try:
        for nodes in (40, 256, 700):
            uf.set_chunk_nodes(nodes)
            d, _, _ = uf.dm(emb, "weighted_normalized", "fp32")
            assert torch.equal(d, full), nodes
    finally:
        uf.set_chunk_nodes(0)
    buf = torch.zeros_like(full)
    s = n // 2
    for b, e in ((0, s // 3), (s // 3, s - s // 4), (s - s // 4, s)):
        uf.dm_stripes(emb, "weighted_normalized", "fp32", b, e, layout="condensed", out=buf)
    assert torch.equal(buf, full)


@pytest.mark.parametrize("n_tips", [40, 700])
def test_batch_of_edge_sizes_equals_single_calls(n_tips):
    import torch
    tree = synth.gen_tree(n_tips, 0.05, n_tips)
    t = uf.Tree(tree.parent, tree.length)
    tabs = [uf.Table(t, x.indptr, x.tips, x.counts)
            for x in (_table(n, n_tips, 3 * n) for n in (2, 65, 64, 3, 257, 63))]
    want = []
    for tb in tabs:
        d, _, _ = uf.dm(uf.Embedding(t, tb), "weighted_normalized", "fp32", out_dtype=torch.float32)
        want.append(d)
    try:
        for nodes in (0, 48, 300):
            uf.set_chunk_nodes(nodes)
            b = uf.Batch(t, tabs)
            for cfg in ((16, 2, 128), (8, 1, 64), (32, 1, 256)):
                b.set_config(*cfg)
                got = b.run()
                torch.cuda.synchronize()
                for g, w in zip(got, want):
                    assert torch.equal(g[:w.numel()], w), (nodes, cfg)
    finally:
        uf.set_chunk_nodes(0)

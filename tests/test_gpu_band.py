"""The fixed-point band tiles of a split's dense set: matrices whose tiles are all cut
along the branches, and one with whole rounds of tiles before the cut ones, against the
FP64 oracle; chunks and stripe ranges, bit for bit."""
import numpy as np
import pytest

import oracle
import paper_2107_05397_amd as uf
import synth

from ._util import random_rows, table as make_table

pytestmark = pytest.mark.gpu


# 512 workgroups; tiles of 128 samples x 256 stripes: 1, 2 and 6 tiles, and 564
@pytest.mark.parametrize("n,n_tips", [(40, 9), (129, 300), (600, 700), (5900, 24)])
def test_band_tiles_match_oracle(n, n_tips):
    import torch
    rng = np.random.default_rng(n)
    tree = synth.gen_tree(n_tips, 0.05, n)
    table = make_table(random_rows(rng, np.arange(n_tips), n, max_nnz=max(2, n_tips // 2)))
    t = uf.Tree(tree.parent, tree.length)
    emb = uf.Embedding(t, uf.Table(t, table.indptr, table.tips, table.counts))
    # the oracle on all samples, or on the first and last of a large matrix
    pick = np.arange(n) if n < 1000 else np.r_[0:150, n - 150:n]
    rows = [slice(table.indptr[i], table.indptr[i + 1]) for i in pick]
    part = make_table([dict(zip(table.tips[r].tolist(), table.counts[r].tolist())) for r in rows])
    want = oracle.dm(tree, part, "weighted_normalized")
    a, b = np.triu_indices(len(pick), 1)
    at = pick[a] * n - pick[a] * (pick[a] + 1) // 2 + pick[b] - pick[a] - 1
    try:
        uf.set_split_threshold(0.0, "weighted_normalized")     # every branch in the dense set
        full, _, _ = uf.dm(emb, "weighted_normalized", "fp32_split")
        uf.profile_reset()
        uf.profile_enable(True)
        again, _, _ = uf.dm(emb, "weighted_normalized", "fp32_split")
        torch.cuda.synchronize()
        uf.profile_enable(False)
        assert torch.equal(again, full)
        # the fixed-point scale is chosen for a distance error of at most 1e-5
        if uf.profile_read("band_wn_u32")[1]:
            assert np.max(np.abs(full.cpu().numpy()[at] - want)) <= 1e-5
        else:
            pytest.fail("the dense pass did not run in fixed point")
        for nodes in (32, 100):
            uf.set_chunk_nodes(nodes)
            d, _, _ = uf.dm(emb, "weighted_normalized", "fp32_split")
            assert torch.equal(d, full), nodes
        uf.set_chunk_nodes(0)
        buf = torch.zeros_like(full)
        s = n // 2
        for b, e in ((0, s // 3), (s // 3, s)):
            uf.dm_stripes(emb, "weighted_normalized", "fp32_split", b, e, layout="condensed", out=buf)
        assert torch.equal(buf, full)
    finally:
        uf.set_chunk_nodes(0)
        uf.set_split_threshold(None)

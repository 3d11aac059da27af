"""Exact re-rank with the query's branches in LDS: candidate counts around the block's
waves, few and many queries, values in LDS and in scratch, and a tree too large for the
bits (dense rows in scratch), against the oracle's pair distances."""
import numpy as np
import pytest

import oracle
import synth

from ._util import random_rows, table as make_table

pytestmark = pytest.mark.gpu


# (tips, tips per sample, queries, references, candidates)
@pytest.mark.parametrize("n_tips,nnz,nq,nr,k", [
    (40, 12, 1, 5, 1), (40, 12, 3, 40, 15), (33, 9, 2, 300, 100), (700, 60, 90, 17, 16),
    (700, 60, 600, 9, 3),
    (12000, 11900, 2, 3, 3),          # 24,000 branches a sample: values in scratch
    (520000, 200, 2, 4, 4),           # over a million branches: dense rows
])
def test_rerank_matches_oracle(n_tips, nnz, nq, nr, k):
    import torch
    import paper_2107_05397_amd as uf
    rng = np.random.default_rng(n_tips + nq)
    tree = synth.gen_tree(n_tips, 0.05, n_tips)
    rows = random_rows(rng, np.arange(n_tips), nq + nr, max_nnz=nnz)
    t = uf.Tree(tree.parent, tree.length)

    def sparse(part):
        tb = make_table(part)
        return uf.Sparse(uf.Embedding(t, uf.Table(t, tb.indptr, tb.tips, tb.counts)))
    sq, sr = sparse(rows[:nq]), sparse(rows[nq:])
    cand = np.stack([rng.permutation(max(nr, k))[:k] % nr for _ in range(nq)]).astype(np.int32)
    got = uf.rerank(sq, sr, torch.arange(nq, dtype=torch.int32, device="cuda"),
                    torch.tensor(cand, device="cuda")).cpu().numpy()
    pick = rng.permutation(nq)[:20]
    pairs = [(int(q), nq + int(r)) for q in pick for r in cand[q]]
    want = oracle.dm_pairs(tree, make_table(rows), pairs, "weighted_normalized").reshape(len(pick), k)
    # FP64 sums of at most K terms each: 8 K eps on a quotient of at most 1
    assert np.max(np.abs(got[pick] - want)) <= 8 * min(tree.n_nodes, 40 * nnz) * 2.0 ** -53

"""A pair's re-ranked distance has the same bits whichever queries and candidates it is asked
for with (one to sixteen waves a candidate, blocks of 256 and 1,024 threads)."""
import numpy as np
import pytest

import synth

from ._util import random_rows, table as make_table

pytestmark = pytest.mark.gpu


# lists shorter than one class of entries, of all sixteen classes and of many rounds; and
# values in scratch
@pytest.mark.parametrize("n_tips,nnz", [(60, 9), (700, 200), (20000, 3000), (12000, 11900)])
def test_distance_is_a_function_of_the_pair(n_tips, nnz):
    import torch
    import paper_2107_05397_amd as uf
    rng = np.random.default_rng(n_tips)
    tree = synth.gen_tree(n_tips, 0.05, n_tips)
    t = uf.Tree(tree.parent, tree.length)

    def sparse(n):
        tb = make_table(random_rows(rng, np.arange(n_tips), n, max_nnz=nnz))
        return uf.Sparse(uf.Embedding(t, uf.Table(t, tb.indptr, tb.tips, tb.counts)))
    few = nnz > 5000
    nq, nr = (3, 30) if few else (40, 120)
    sq, sr = sparse(nq), sparse(nr)

    def run(ids, cand):
        return uf.rerank(sq, sr, torch.tensor(ids, dtype=torch.int32, device="cuda"),
                         torch.tensor(np.ascontiguousarray(cand), dtype=torch.int32, device="cuda"))
    ids = np.arange(nq)
    cand = np.stack([rng.permutation(nr) for _ in ids])
    want = run(ids, cand)
    big = np.tile(ids, 600 // nq + 1)                          # more queries than workgroups' share
    assert torch.equal(run(big, cand[big])[:nq], want)
    for k in (1, 3, 5):                                        # many, with few candidates
        assert torch.equal(run(big, cand[big, :k])[:nq], want[:, :k].contiguous()), k
    for k in (1, 2, 3, 5, 9, 16, nr):                          # one query, and all, with k candidates
        assert torch.equal(run(ids, cand[:, :k]), want[:, :k].contiguous()), k
        assert torch.equal(run(ids[:1], cand[:1, :k]), want[:1, :k].contiguous()), k

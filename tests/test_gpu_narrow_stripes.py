"""A few stripes of a large matrix run on the tiles that hold them alone: the same bits as the
whole matrix's stripes, at its first, last and middle ones."""
import numpy as np
import pytest

import paper_2107_05397_amd as uf
import synth

from ._util import random_rows, table as make_table

pytestmark = pytest.mark.gpu


# one block and its edges, several; from 4,096 samples on the weighted tiles of all stripes are
# wider than those of a few
@pytest.mark.parametrize("n", [5, 64, 129, 700, 1501, 4500])
@pytest.mark.parametrize("variant,precision", [("weighted", "fp64"), ("weighted", "fp32"),
                                               ("unweighted", "fp64"), ("unweighted", "fp32")])
def test_few_stripes_equal_all(n, variant, precision):
    import torch
    rng = np.random.default_rng(n)
    tree = synth.gen_tree(80, 0.05, n)
    table = make_table(random_rows(rng, np.arange(80), n, max_nnz=20))
    t = uf.Tree(tree.parent, tree.length)
    emb = uf.Embedding(t, uf.Table(t, table.indptr, table.tips, table.counts))
    s = n // 2
    full, _ = uf.dm_stripes(emb, variant, precision, 0, s)
    for b, e in {(0, 1), (s - 1, s), (s // 2, s // 2 + 1), (0, min(s, 70)), (max(0, s - 65), s),
                 (s // 3, min(s, s // 3 + 130)), (s // 4, s // 2)}:
        if b < e:
            part, _ = uf.dm_stripes(emb, variant, precision, b, e)
            assert torch.equal(part, full[b:e]), (b, e)

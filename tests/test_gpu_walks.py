"""The walks over a sample's branches with rows at the edge of what is kept in LDS (1,024
entries) and past it, and the projection at its widest output."""
import numpy as np
import pytest

import oracle
import paper_2107_05397_amd as uf
import synth
from oracle import placement as op

from ._util import table as make_table

pytestmark = pytest.mark.gpu

N_TIPS = 1700


def _table():
    rng = np.random.default_rng(4)
    rows = []
    for m in (1, 2, 255, 1023, 1024, 1025, 1300, N_TIPS):
        tips = rng.permutation(N_TIPS)[:m]
        rows.append({int(t): int(c) for t, c in zip(tips, rng.integers(1, 900, m))})
    return make_table(rows)


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_split"])
def test_long_rows_match_oracle(precision):
    tree, table = synth.gen_tree(N_TIPS, 0.05, 11), _table()
    t = uf.Tree(tree.parent, tree.length)
    emb = uf.Embedding(t, uf.Table(t, table.indptr, table.tips, table.counts))
    want = oracle.dm(tree, table, "weighted_normalized")
    got, _, _ = uf.dm(emb, "weighted_normalized", precision)
    # at most K terms, each rounded, over a bound of their sum; the split's dense part is
    # in fixed point with a distance error of at most 1e-5
    tol = {"fp64": 6 * tree.n_nodes * 2.0 ** -53, "fp32": (tree.n_nodes + 2) * 2.0 ** -24,
           "fp32_split": 1e-5 + (tree.n_nodes + 2) * 2.0 ** -24}[precision]
    assert np.max(np.abs(got.cpu().numpy() - want)) <= tol


@pytest.mark.parametrize("out_dim,per_node", [(64, 1), (4096, 4), (8192, 16)])
def test_projection_of_long_rows(out_dim, per_node):
    tree, table = synth.gen_tree(N_TIPS, 0.05, 11), _table()
    t = uf.Tree(tree.parent, tree.length)
    emb = uf.Embedding(t, uf.Table(t, table.indptr, table.tips, table.counts))
    dims, signs = synth.sparse_projection(tree.n_nodes, out_dim=out_dim, per_node=per_node, seed=5)
    got = uf.project(t, emb, dims, signs, out_dim=out_dim).float().cpu().numpy().astype(np.float64)
    want = op.project(tree, table, dims, signs, out_dim)
    # one BF16 rounding, and a rounding to 2^-40 for each of at most K terms
    assert np.all(np.abs(got - want) <= np.abs(want) * 2.0 ** -8 + tree.n_nodes * 2.0 ** -41)

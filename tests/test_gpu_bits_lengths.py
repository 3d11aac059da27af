"""Unweighted distances and the rounding of branch lengths to the digits of the product on
presence bits: equal samples are at distance 0, samples that differ on little keep their
relative accuracy, and lengths far below the longest are not lost, whatever their range."""
import dataclasses

import numpy as np
import pytest

import oracle
import paper_2107_05397_amd as uf
import synth

from ._util import random_rows, table as make_table

pytestmark = pytest.mark.gpu


def _distances(tree, table, precision):
    import torch  # noqa: F401
    t = uf.Tree(tree.parent, tree.length)
    emb = uf.Embedding(t, uf.Table(t, table.indptr, table.tips, table.counts))
    return uf.dm(emb, "unweighted", precision)[0].cpu().numpy()


def _square(cond, n):
    d = np.zeros((n, n))
    d[np.triu_indices(n, 1)] = cond
    return d + d.T


# 0.1 on every branch beside one (of tip 0, which no sample holds) of 3, 50, 1e4 and 1e9: all
# digits; FP64 without them, and FP32 with more; both; FP32 without them
@pytest.mark.parametrize("longest", [3.0, 50.0, 1e4, 1e9])
@pytest.mark.parametrize("precision,eps", [("fp64", 2.0 ** -53), ("fp32", 2.0 ** -24), ("mfma", 2.0 ** -24)])
def test_equal_short_lengths(longest, precision, eps):
    import torch
    rng = np.random.default_rng(3)
    tree = synth.gen_tree(900, 0.05, 3)
    short = float(np.float32(0.1))
    hi = float(torch.tensor(short).to(torch.bfloat16))
    lo = float(torch.tensor(short - hi).to(torch.bfloat16))
    length = np.where(np.arange(tree.n_nodes) == 0, longest, short)
    rows = random_rows(rng, np.arange(1, 900), 130, max_nnz=150)
    for k in range(3):                                         # equal samples, two blocks apart
        rows[127 + k] = dict(rows[k])
    table = make_table(rows)
    work = dataclasses.replace(tree, length=np.where(np.arange(tree.n_nodes) == 0, longest,
                                                     hi + lo if precision == "mfma" else short))
    want = oracle.dm(work, table, "unweighted")
    got = _distances(dataclasses.replace(tree, length=length), table, precision)
    square = _square(got, 130)
    # all sums are multiples of one length: digits change both sums alike, and d by their own
    # rounding alone; without digits, by sums of K equal lengths in the type
    bound = 6 * tree.n_nodes * eps if longest == 1e9 or (precision == "fp64" and longest > 3) else 4 * eps
    assert np.max(np.abs(got - want)) <= bound
    if bound == 4 * eps:
        assert square[0, 127] == 0 and square[1, 128] == 0 and square[2, 129] == 0


# lengths spread over a range, and one sample of a single tip: still within the digits' bound
# (2^-50 and 2^-22) beside the oracle's own sums and one rounded result
@pytest.mark.parametrize("n_tips", [60, 5000])
@pytest.mark.parametrize("precision,bound", [("fp64", 2.0 ** -50), ("fp32", 2.0 ** -22)])
def test_shallow_sample(n_tips, precision, bound):
    rng = np.random.default_rng(n_tips)
    tree = synth.gen_tree(n_tips, 0.05, n_tips)
    tree = dataclasses.replace(tree, length=tree.length.astype(np.float32).astype(np.float64))
    rows = random_rows(rng, np.arange(n_tips), 70, max_nnz=n_tips // 4)
    rows[5] = {int(rng.integers(n_tips)): 7}
    rows[66] = dict(rows[4])
    table = make_table(rows)
    want = oracle.dm(tree, table, "unweighted")
    got = _distances(tree, table, precision)
    assert np.max(np.abs(got - want)) <= bound + 8 * tree.n_nodes * 2.0 ** -53
    assert _square(got, 70)[4, 66] == 0


# samples of 3,000 tips that differ on one tip each: d ~ 1e-4 of exact integers
def test_close_samples():
    tree = synth.gen_tree(6000, 0.05, 9)
    tree = dataclasses.replace(tree, length=np.ldexp(np.floor(np.ldexp(tree.length, 40)), -40))
    base = np.random.default_rng(1).permutation(6000)
    table = make_table([{int(t): 1 for t in np.r_[base[:3000], base[3000 + s]]} for s in range(70)])
    want = oracle.dm(tree, table, "unweighted")
    got = _distances(tree, table, "fp64")
    # lengths on a grid of 2^-40 are held exactly: both sums are exact, with one rounding each
    # and one of the quotient; the oracle adds up to K terms in each
    assert np.all(np.abs(got - want) <= (2 * tree.n_nodes + 4) * 2.0 ** -53 * want)

"""The batch's configuration: what a tuning run times differs, and wgs_per_cu, which records
may name, changes nothing."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _batch(uf, sizes, n_tips, nnz):
    tree = synth.gen_tree(n_tips, 0.05, seed=5)
    t = uf.Tree(tree.parent, tree.length)
    tabs = []
    for r, n in enumerate(sizes):
        x = synth.gen_table_uniform(n, np.arange(n_tips), nnz, seed=70 + r)
        tabs.append(uf.Table(t, x.indptr, x.tips, x.counts))
    return uf.Batch(t, tabs)


def test_tuned_configuration_is_one_of_the_distinct_ones(tmp_path):
    import torch
    import paper_2107_05397_amd as uf
    largest = {(8, 64): 5, (8, 128): 3, (8, 256): 2, (16, 64): 3, (16, 128): 2, (16, 256): 2,
               (32, 64): 1, (32, 128): 1, (32, 256): 1}
    for sizes in ((700, 500), (4200,)):
        b = _batch(uf, sizes, 400, 60)
        want = [o.clone() for o in b.run()]
        tile = b.config()[3]
        assert b.autotune(str(tmp_path / "tune.json")) > 0
        ks, w, _, ts = b.config()
        assert w == largest[ks, ts]
        assert ts == tile or len(sizes) > 1        # wide tables alone: no tile to choose
        for w in range(1, largest[8, 64] + 1):
            b.set_config(8, w, 64)
            assert all(torch.equal(g, o) for g, o in zip(b.run(), want))

"""A batch's graph given up (new configuration, other outputs, other precision, the batch
freed) while a replay of it may still run: every replay's results are whole."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_graph_given_up_while_in_flight():
    import torch
    import paper_2107_05397_amd as uf
    tree = synth.gen_tree(2000, 0.05, seed=3)
    t = uf.Tree(tree.parent, tree.length)
    tabs = []
    for r, n in enumerate((700, 450, 90)):
        x = synth.gen_table_zipf(n, np.arange(2000), 200, seed=40 + r)
        tabs.append(uf.Table(t, x.indptr, x.tips, x.counts))
    b = uf.Batch(t, tabs)
    want = [o.clone() for o in b.run()]
    others = [torch.zeros_like(o) for o in b.outputs()]
    torch.cuda.synchronize()
    got = []
    for cfg in ((8, 2, 64), (16, 1, 256), (32, 1, 128), (16, 2, 128)):
        b.set_config(*cfg)                       # (each time just after a replay was enqueued)
        for outs in (b.outputs(), others):
            for o in outs:
                o.zero_()
            got += [o.clone() for o in b.run(outs=outs)]
    b.set_precision("fp32_split")
    b.set_precision("fp32")
    got += [o.clone() for o in b.run()]
    b.close()
    torch.cuda.synchronize()
    for k, g in enumerate(got):
        w = want[k % len(want)]
        assert torch.equal(g[:w.numel()], w), k

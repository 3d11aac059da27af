"""Mantel permutations with S's rows kept in LDS: one and several rows per block, the
permutations in shares, and rows of indices that are no permutation (which the general
kernel takes) against a direct sum."""
import numpy as np
import pytest

from oracle import mantel as om

pytestmark = pytest.mark.gpu


def _matrices(n, seed):
    rng = np.random.default_rng(seed)
    p = rng.normal(size=(n, 5))
    iu = np.triu_indices(n, 1)
    x = np.linalg.norm(p[iu[0]] - p[iu[1]], axis=1)
    return x, x + rng.normal(scale=0.5, size=x.size)


# one row per block (up to 256 samples), two and three, the last block with fewer; one
# permutation, fewer than a block's waves, several shares
@pytest.mark.parametrize("n,n_perm", [(3, 1), (64, 200), (256, 17), (257, 40), (513, 5), (700, 33)])
def test_rows_in_lds_match_oracle(n, n_perm):
    import torch
    import paper_2107_05397_amd as uf
    x, y = _matrices(n, n)
    rng = np.random.default_rng(n + 1)
    perms = np.stack([rng.permutation(n) for _ in range(n_perm)]).astype(np.int32)
    perms[n_perm // 2] = np.arange(n)
    st, p, ps = uf.mantel(torch.tensor(x, device="cuda"), torch.tensor(y, device="cuda"), n, "pearson",
                          torch.tensor(perms, device="cuda"))
    st_o, p_o, ps_o = om.mantel(x, y, n, "pearson", perms)
    assert abs(st - st_o) <= 1e-12 and np.allclose(ps, ps_o, atol=1e-12) and p == p_o
    assert ps[n_perm // 2] == st


def test_rows_that_are_no_permutation():
    import torch
    import paper_2107_05397_amd as uf
    n = 90
    x, y = _matrices(n, 4)
    maps = np.stack([np.random.default_rng(k).permutation(n) for k in range(20)]).astype(np.int32)
    maps[7] = np.random.default_rng(99).integers(0, n, n)      # samples twice and not at all
    _, _, ps = uf.mantel(torch.tensor(x, device="cuda"), torch.tensor(y, device="cuda"), n, "pearson",
                         torch.tensor(maps, device="cuda"))
    xs, ys = (v - v.mean() for v in (x, y))
    xs, ys = xs / np.linalg.norm(xs), ys / np.linalg.norm(ys)
    iu = np.triu_indices(n, 1)
    s = np.zeros((n, n))
    s[iu] = xs
    s = s + s.T                                                # 0 on the diagonal
    want = [float((s[m[iu[0]], m[iu[1]]] * ys).sum()) for m in maps]
    assert np.allclose(ps, want, atol=1e-12)

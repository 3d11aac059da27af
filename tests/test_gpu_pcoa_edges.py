"""PCoA at the edges of its tiles, column groups and partial sums: points in a space of known
dimension, whose nonzero eigenvalues are those of the centred points' Gram matrix and whose
coordinates reproduce every distance, with more columns than the rank (dependent columns)."""
import numpy as np
import pytest

import paper_2107_05397_amd as uf

pytestmark = pytest.mark.gpu


# rows: below, at and past the tiles of 16 and 32, several Gram tiles, several tiles a Gram
# block (past 8,192); columns: each group of 16, its edge; at most as many as samples
@pytest.mark.parametrize("n,rank,cols", [(2, 1, 1), (3, 2, 3), (15, 4, 9), (16, 4, 16), (17, 3, 17),
                                         (33, 5, 33), (64, 5, 48), (65, 6, 32), (129, 2, 20),
                                         (500, 7, 16), (8300, 4, 18)])
@pytest.mark.parametrize("means", [True, False])
def test_points_are_recovered(n, rank, cols, means):
    import torch
    rng = np.random.default_rng(n + cols)
    x = rng.standard_normal((n, rank)) * 0.8 ** np.arange(rank)
    t = torch.as_tensor(x, device="cuda")
    i, j = torch.triu_indices(n, n, 1, device="cuda")
    d = (t[i] - t[j]).pow(2).sum(1).sqrt()
    kw = {}
    if means:
        sq = (t - t.mean(0)).pow(2).sum(1)
        r = -0.5 * (sq + sq.mean())                            # row means of -d^2/2
        kw = dict(row_means=r, grand_mean=r.mean().reshape(1))
    omega = torch.as_tensor(rng.standard_normal((n, cols)), device="cuda")
    coords, vals, trace = uf.pcoa(d, n, rank, omega, power_iters=1, **kw)
    torch.cuda.synchronize()
    want = np.linalg.svd(x - x.mean(0), compute_uv=False) ** 2
    # sums of n terms and products of orthonormal bases, each rounded: n eps of the largest
    tol = 1e-13 * max(n, 100) * want[0]
    got = np.asarray(vals)[:rank]
    assert np.max(np.abs(got - want[:rank])) <= tol
    assert abs(trace - want.sum()) <= tol * rank
    c = coords[:, :rank]
    back = (c[i] - c[j]).pow(2).sum(1)
    assert float((back - d * d).abs().max()) <= tol * 10


def test_equal_points_and_not_a_number():
    import torch
    n = 40
    omega = torch.randn(n, 5, dtype=torch.float64, device="cuda")
    for fill in (0.0, float("nan")):
        d = torch.full((n * (n - 1) // 2,), fill, dtype=torch.float64, device="cuda")
        coords, vals, _ = uf.pcoa(d, n, 3, omega, power_iters=2)
        assert np.all(np.asarray(vals) == 0.0) and float(coords.abs().max()) == 0.0

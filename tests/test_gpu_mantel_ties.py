"""Mantel permutations that leave the first matrix unchanged: the same terms, so the observed
statistic bit for bit, and all of them counted by the p-value's comparisons."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _classes(n, kind):
    """A class per sample; samples of one class are interchangeable."""
    if kind == "groups":
        return np.arange(n) * 2 // n, np.array([[0.0, 1.0], [1.0, 0.0]])
    k = (n + 1) // 2                                           # every sample twice (one once)
    p = np.random.default_rng(n).normal(size=(k, 4))
    return np.arange(n) % k, np.linalg.norm(p[:, None] - p[None], axis=2)


# one row of the matrix per block (up to 256 samples), three (not a whole set of four), eight
@pytest.mark.parametrize("n", [4, 12, 60, 256, 700, 2000])
@pytest.mark.parametrize("kind", ["groups", "duplicates"])
@pytest.mark.parametrize("method", ["pearson", "spearman"])
def test_relabelled_equals_observed(n, kind, method):
    import torch
    import paper_2107_05397_amd as uf
    rng = np.random.default_rng(n)
    cls, between = _classes(n, kind)
    iu = np.triu_indices(n, 1)
    x = between[cls[iu[0]], cls[iu[1]]]
    y = rng.random(x.size)
    perms = []
    for _ in range(40):
        p = np.arange(n)
        for c in np.unique(cls):
            at = np.flatnonzero(cls == c)
            p[at] = rng.permutation(at)
        if kind == "groups" and n % 2 == 0 and rng.random() < 0.5:
            p = np.roll(p, n // 2)                             # the groups exchanged
        perms.append(p)
    perms = np.stack(perms).astype(np.int32)
    for alternative in ("two-sided", "greater", "less"):
        st, p, ps = uf.mantel(torch.tensor(x, device="cuda"), torch.tensor(y, device="cuda"), n, method,
                              torch.tensor(perms, device="cuda"), alternative=alternative)
        assert np.all(np.asarray(ps) == st), int(np.sum(np.asarray(ps) != st))
        assert p == 1.0

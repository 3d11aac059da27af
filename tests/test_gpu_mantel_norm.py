"""Mantel: the norms of long vectors, summed from many parts."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [400, 4000])
def test_norm_of_two_spikes(n):
    """x with itself is at 1.  Two values of +-1 and the rest +-a (their mean 0), a so small that
    4,096 of their squares come to 0.45 ulp of the squares' sum: added one part after the other
    each would be lost (4,000 samples: 1,953 parts, 2e-13).

    Bound: every value passes at most 32 additions in its thread and 8 between threads, or in
    the product ceil(n / 64) + 6 and ceil(n / 256) + 8, and log2 of the number of parts; with
    3 roundings in each vector and in the norms the relative errors add up to the count of
    these, in units of 2^-53."""
    import torch
    import paper_2107_05397_amd as uf
    m = n * (n - 1) // 2
    a = np.sqrt(0.45 * 2.0**-51 / 4096)
    x = np.where(np.arange(m) % 2 == 0, a, -a)
    x[0], x[1] = 1.0, -1.0
    xd = torch.tensor(x, device="cuda")
    perms = torch.arange(n, dtype=torch.int32, device="cuda").repeat(2, 1)
    r, _, ps = uf.mantel(xd, xd, n, "pearson", perms)
    depth = 40 + 13 + (n + 63) // 64 + 6 + (n + 255) // 256 + 8 + 12
    assert abs(r - 1.0) <= depth * 2.0**-53, r - 1.0
    assert np.all(ps == r)

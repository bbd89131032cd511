"""k-means assignment where the split product's bound leaves many points open:
isotropic rows, unit rows with a common mean, rows far from the origin, and
centroids that are copies of each other (exact ties, decided by the sequential
sums).  More and fewer queued points than the 16-row and 32-row workgroups
take, columns past one sweep of a workgroup, dimensions with and without wide
loads; equal to the FP64 oracle everywhere."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _rows(kind, n, d, g):
    X = g.standard_normal((n, d))
    if kind == "unit":
        X += 1.5 * g.standard_normal((1, d))
        X /= np.linalg.norm(X, axis=1, keepdims=True)
    elif kind == "offset":
        X = 100.0 + X
    elif kind == "far":
        X = 3000.0 + X
    return X.astype(np.float32)


@pytest.mark.parametrize("kind", ["iso", "unit", "offset", "far", "copies"])
@pytest.mark.parametrize("n,d,C", [(5, 16, 3), (300, 64, 33), (1500, 100, 513), (1500, 99, 700),
                                   (20000, 64, 40), (9000, 33, 64), (700, 768, 300), (40, 7, 1100)])
def test_equal_to_the_oracle(kind, n, d, C):
    import torch
    from paper_2205_00970_amd import lider
    g = np.random.default_rng(n + d + C)
    X = _rows(kind, n, d, g)
    cent = _rows(kind, C, d, g)
    if C <= n:  # means of a few rows each, as in the middle of a k-means
        cent = np.stack([X[j::C][:3].mean(axis=0) for j in range(C)]).astype(np.float32)
    if kind == "copies":
        cent[C // 2:] = cent[:C - C // 2]
    want = oracle.kmeans_assign(X, cent)
    got = lider.kmeans_assign(torch.from_numpy(X).cuda(), torch.from_numpy(cent).cuda()).cpu().numpy()
    assert np.array_equal(got, want)
    buf = torch.empty(n * d + 1, device="cuda")  # rows at addresses that are not multiples of 16 bytes
    buf[1:] = torch.from_numpy(X.reshape(-1)).cuda()
    got = lider.kmeans_assign(buf[1:].view(n, d), torch.from_numpy(cent).cuda()).cpu().numpy()
    assert np.array_equal(got, want)


@pytest.mark.parametrize("copies", [2, 3, 40, 200])
@pytest.mark.parametrize("n,d,C", [(300, 32, 400), (9000, 20, 400), (100, 33, 1200)])
def test_many_equal_centroids(n, d, C, copies):
    """Ties of few centroids (listed) and of more than a list holds (all summed)."""
    import torch
    from paper_2205_00970_amd import lider
    g = np.random.default_rng(n + copies)
    X = g.standard_normal((n, d)).astype(np.float32)
    cent = np.repeat(g.standard_normal((C // copies + 1, d)), copies, axis=0)[:C].astype(np.float32)
    cent = cent[g.permutation(C)]
    got = lider.kmeans_assign(torch.from_numpy(X).cuda(), torch.from_numpy(cent).cuda()).cpu().numpy()
    assert np.array_equal(got, oracle.kmeans_assign(X, cent))

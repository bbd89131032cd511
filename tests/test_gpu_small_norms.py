"""Queries whose elements' squares vanish in fp32 (below 2^-75) or lose bits
there: their norms still bound the error of the split products, so many
near-duplicate rows are ranked, and clusters routed, as without them.  The
split window scores against the fp32 windows bit for bit, the routed clusters
against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2205_00970_amd import datagen

pytestmark = pytest.mark.gpu


def _near(X, at, g):
    """Rows `at` become copies of the first with elements changed by up to 2^-17 of them."""
    X[at] = X[at[0]] * (1.0 + 2.0**-20 * g.integers(-8, 9, (at.size, X.shape[1]))).astype(np.float32)


@pytest.mark.parametrize("H", [1, 3])
@pytest.mark.parametrize("scale", [1.0, 2e-19, 1e-21, 1e-23, 1e-25])
def test_near_duplicate_rows(H, scale):
    import torch
    from paper_2205_00970_amd import lider
    n, d, C = 20000, 64, 70
    X, lab, Q, _ = datagen.tiny(n=n, d=d, ncomp=C, nq=1500, seed=110, qseed=111)
    g = np.random.default_rng(112)
    for j in (3, 4):
        at = np.nonzero(lab == j)[0][:60]
        _near(X, at, g)
        Q[100 * j:100 * j + 40] = X[at[0]] + 0.01 * Q[100 * j:100 * j + 40]
    X = (X * np.float32(1e6)).astype(np.float32)  # the margin's absolute terms are far below the scores' error
    Q = (Q * np.float32(scale)).astype(np.float32)
    A, b = datagen.lsh_params(6, d, 1e6, seed=113, n_arrays=H)
    gi = lider.Index(torch.from_numpy(X).cuda(), C, 6, 1e6, 8, (A, b), n_arrays=H,
                     assignment=torch.from_numpy(lab).cuda())
    Qd = torch.from_numpy(Q).cuda()
    a = gi.search(Qd, 10, 4, 100, r1=C)
    e = gi.search(Qd, 10, 4, 100, r1=C, tile_rows=128, pass_pairs=128)
    assert torch.equal(a[0], e[0])
    assert torch.equal(a[1].view(torch.int32), e[1].view(torch.int32))


@pytest.mark.parametrize("d,c", [(64, 1), (64, 3), (100, 1), (100, 3)])
@pytest.mark.parametrize("scale", [1.0, 1e-21, 1e-23])
def test_routing_between_near_duplicate_centroids(d, c, scale):
    import torch
    from paper_2205_00970_amd import lider
    n, C = 4000, 64  # 40 clusters with nearly the same centroid
    g = np.random.default_rng(114 + d)
    mu = g.standard_normal((C, d))
    mu[:40] = 2.0 * mu[0] * (1.0 + 2.0**-20 * g.integers(-8, 9, (40, d)))
    mu *= 1e6
    lab = (np.arange(n) % C).astype(np.int32)
    X = mu[lab].astype(np.float32)
    Q = ((mu[0] / 1e6 + 0.05 * g.standard_normal((60, d))) * scale).astype(np.float32)
    A, b = datagen.lsh_params(4, d, 1e6, seed=115)
    gi = lider.Index(torch.from_numpy(X).cuda(), C, 4, 1e6, 8, (A, b), assignment=torch.from_numpy(lab).cuda())
    oi = oracle.Index(X, C, A, b, 4, 1e6, 8, assignment=lab)
    _, _, dbg = gi.search(torch.from_numpy(Q).cuda(), 10, c, 64, r1=C, debug=True)
    _, _, odbg = oi.search(Q, 10, c, 64, C, debug=True)
    assert np.array_equal(np.sort(dbg["routed"].cpu().numpy(), axis=1), np.sort(odbg["routed"], axis=1))

"""The k-means assignment where |x|^2 and |mu|^2 fit fp32 and 2 x.mu does not:
the nearest centroid is still the FP64 oracle's."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C", [2, 40, 300])
@pytest.mark.parametrize("d", [4, 33, 64])
def test_overflowing_products(C, d):
    import torch
    from paper_2205_00970_amd import lider
    g = np.random.default_rng(C + d)
    u = g.standard_normal(d)
    u /= np.linalg.norm(u)
    X = np.outer(g.uniform(1.30e19, 1.36e19, 500), u).astype(np.float32)
    # 2 x.mu past 3.4e38 for the long centroids only, the short ones nearer
    cent = np.outer(np.where(np.arange(C) % 2 == 0, 1.7e19, 1.24e19) * g.uniform(0.99, 1.0, C), u).astype(np.float32)
    want = oracle.kmeans_assign(X, cent)
    assert (want % 2 == 1).all()
    got = lider.kmeans_assign(torch.from_numpy(X).cuda(), torch.from_numpy(cent).cuda()).cpu().numpy()
    assert np.array_equal(got, want)

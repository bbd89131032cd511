"""Farthest-first seeding over short lists: dimensions with and without wide
loads, several lists, exact ties and duplicate rows (more candidates than a
round decides, and rows all at distance zero), bounds too wide for a list,
against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2205_00970_amd import datagen

pytestmark = pytest.mark.gpu


def _rows(kind, n, d):
    g = np.random.default_rng(n + d)
    if kind == "spread":  # no clusters: the lists run out often
        return g.standard_normal((n, d)).astype(np.float32)
    if kind == "grid":  # whole numbers: many exactly equal distances
        return g.integers(0, 3, (n, d)).astype(np.float32)
    if kind == "copies":  # 20 distinct rows
        return g.standard_normal((20, d)).astype(np.float32)[np.arange(n) % 20]
    if kind == "offset":  # distances far below the rows' norms: the product's bounds are too wide
        return (1000.0 + g.standard_normal((n, d))).astype(np.float32)
    X = g.standard_normal((12, d))[g.integers(0, 12, n)] + 0.05 * g.standard_normal((n, d))
    X[::97] *= 5.0  # outliers
    return X.astype(np.float32)


@pytest.mark.parametrize("kind,n,d,C,shift", [("spread", 6000, 64, 300, 0), ("spread", 5000, 33, 120, 0),
                                              ("spread", 3000, 8, 1500, 1), ("grid", 4000, 6, 60, 0),
                                              ("copies", 2000, 36, 30, 0), ("blobs", 20000, 48, 40, 0),
                                              ("blobs", 17, 100, 17, 0), ("spread", 2, 4, 2, 0),
                                              ("offset", 3000, 32, 40, 0), ("offset", 2500, 19, 20, 0)])
def test_seeds_equal_the_oracle(kind, n, d, C, shift):
    import torch
    from paper_2205_00970_amd import lider
    X = _rows(kind, n, d)
    buf = torch.empty(n * d + shift, device="cuda")  # shift: rows not at multiples of 16 bytes
    buf[shift:] = torch.from_numpy(X.reshape(-1)).cuda()
    first = n // 3
    A, b = datagen.lsh_params(4, d, 2.0, seed=5)
    init = np.array([first], np.int64)
    gi = lider.Index(buf[shift:].view(n, d), C, 4, 2.0, 4, (A, b), kmeans_init=init, kmeans_iters=1,
                     seeding="farthest")
    ids = oracle.kmeans_seed_farthest(X, C, first)
    ref = oracle.kmeans_assign(X, X[ids])  # one Lloyd step from the oracle's seeds
    assert np.array_equal(gi.export("assign"), ref)

"""Farthest-first seeding over rows whose squares or products overflow fp32:
the picks stay those of the FP64 oracle.  Rows of moderate norm with one so
large that its square sum and its product with every centroid overflow, in a
direction close to theirs; rows whose square sums fit while products do not;
and the same with a row that holds a NaN, which is never picked."""
import numpy as np
import pytest

import oracle
from paper_2205_00970_amd import datagen

pytestmark = pytest.mark.gpu


def _rows(kind, n, d):
    g = np.random.default_rng(n + d)
    X = 1.0 + 0.2 * g.standard_normal((n, d))
    X /= np.linalg.norm(X, axis=1, keepdims=True)
    if kind == "one_large":  # |x| |mu| = 1e40 in nearly the same direction
        X *= 1e15
        X[77] *= 1e10
        X[78] *= 1e9
    else:  # |x|^2 < 3.4e38 < 2 |x| |mu|
        X *= g.uniform(1.2e19, 1.8e19, (n, 1))
    return X.astype(np.float32)


@pytest.mark.parametrize("kind", ["one_large", "all_large"])
@pytest.mark.parametrize("n,d,C", [(3000, 64, 12), (2500, 19, 150)])
def test_picks_equal_the_oracle(kind, n, d, C):
    import torch
    from paper_2205_00970_amd import lider
    X = _rows(kind, n, d)
    first = n // 3
    A, b = datagen.lsh_params(4, d, 2.0, seed=5)
    gi = lider.Index(torch.from_numpy(X).cuda(), C, 4, 2.0, 4, (A, None), hash_kind="sign",
                     kmeans_init=np.array([first], np.int64), kmeans_iters=1, seeding="farthest")
    ids = oracle.kmeans_seed_farthest(X, C, first)
    if kind == "one_large":
        assert 77 in ids
    assert np.array_equal(gi.export("assign"), oracle.kmeans_assign(X, X[ids]))

"""Split window scores where lists are long: groups of equal rows, past a list's
room, in a few clusters (their queries' windows are scored again in fp32, the
others keep their lists), in every cluster, and a row whose norm widens the
bound past every score (the index then keeps the fp32 windows); with block
keys, several arrays, few candidates and a batch with one such query.  Ids and
scores equal the search with an explicit rerank shape bit for bit."""
import numpy as np
import pytest

from paper_2205_00970_amd import datagen

pytestmark = pytest.mark.gpu


def _index(kind, H, d=96, n=20000, C=70):
    import torch
    from paper_2205_00970_amd import lider
    X, lab, Q, _ = datagen.tiny(n=n, d=d, ncomp=C, nq=1500, seed=120, qseed=121)
    groups = {"few": (3, 4, 9), "all": range(C), "large": ()}[kind]
    for t, j in enumerate(groups):
        at = np.nonzero(lab == j)[0][:150]
        X[at] = X[at[0]]
        Q[20 * t:20 * t + 20] = X[at[0]] + 0.01 * Q[20 * t:20 * t + 20]
    if kind == "large":
        X[77] *= 1e4
    A, b = datagen.lsh_params(6, d, 1.0, seed=122, n_arrays=H)
    gi = lider.Index(torch.from_numpy(X).cuda(), C, 6, 1.0, 8, (A, b), n_arrays=H,
                     assignment=torch.from_numpy(lab).cuda())
    return gi, torch.from_numpy(Q).cuda()


@pytest.mark.parametrize("H", [1, 2])
@pytest.mark.parametrize("kind", ["few", "all", "large"])
def test_equal_to_the_fp32_windows(kind, H):
    import torch
    gi, Q = _index(kind, H)
    for k, c, r in ((10, 4, 100), (10, 16, 286), (16, 8, 400), (3, 3, 64)):
        a = gi.search(Q, k, c, r, r1=70)
        e = gi.search(Q, k, c, r, r1=70, tile_rows=128, pass_pairs=128)
        assert torch.equal(a[0], e[0]), (k, c, r)
        assert torch.equal(a[1].view(torch.int32), e[1].view(torch.int32)), (k, c, r)


def test_one_query_with_a_long_list():
    import torch
    gi, Q = _index("few", 1)
    Q = Q[60:].clone()  # no query near a group
    Q[700] = 0.0
    for k, c, r in ((10, 16, 286), (1, 4, 100)):
        a = gi.search(Q, k, c, r, r1=70)
        e = gi.search(Q, k, c, r, r1=70, tile_rows=128, pass_pairs=128)
        assert torch.equal(a[0], e[0]) and torch.equal(a[1].view(torch.int32), e[1].view(torch.int32))

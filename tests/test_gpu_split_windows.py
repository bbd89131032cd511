"""Split window scores (many pairs per tile, short result lists): ids and
scores equal, bit for bit, the search with an explicit rerank shape, which
scores every window by the fp32 product; over arrays, expansion, dimensions,
k around the limit, exact ties past the list's room, and queries without a
margin (zero, huge, infinite, NaN)."""
import numpy as np
import pytest

from paper_2205_00970_amd import datagen

pytestmark = pytest.mark.gpu


def _index(n, d, C, H=1, kind="e2lsh", copies=0, seed=0):
    import torch
    from paper_2205_00970_amd import lider
    X, lab, Q, _ = datagen.tiny(n=n, d=d, ncomp=C, nq=1500, seed=70 + seed, qseed=71 + seed)
    if copies:  # equal rows in one cluster: equal scores past the list's room
        at = np.nonzero(lab == 3)[0][:copies]
        X[at] = X[at[0]]
        Q[:40] = X[at[0]] + 0.01 * Q[:40]
    if kind == "sign":
        X, Q = datagen.normalize_rows(X), datagen.normalize_rows(Q)
    A, b = datagen.lsh_params(6, d, 1.0, seed=72, n_arrays=H)
    gi = lider.Index(torch.from_numpy(X).cuda(), C, 6, 1.0, 8, (A, None if kind == "sign" else b),
                     assignment=torch.from_numpy(lab).cuda(), hash_kind=kind, n_arrays=H)
    return gi, torch.from_numpy(Q).cuda()


def _same(gi, Q, k, c, r, **kw):
    import torch
    a = gi.search(Q, k, c, r, **kw)
    b = gi.search(Q, k, c, r, tile_rows=128, pass_pairs=128, **kw)
    assert torch.equal(a[0], b[0])
    assert torch.equal(a[1].view(torch.int32), b[1].view(torch.int32))


@pytest.mark.parametrize("d,H,kind,B", [(96, 1, "e2lsh", 0), (32, 1, "e2lsh", 0), (128, 3, "e2lsh", 0),
                                        (64, 1, "sign", 3), (160, 2, "sign", 2)])
@pytest.mark.parametrize("copies", [0, 150])
def test_equal_to_the_fp32_windows(d, H, kind, B, copies):
    gi, Q = _index(20000, d, 70, H, kind, copies)
    for k, c, r in ((10, 4, 100), (1, 3, 64), (16, 8, 256), (17, 4, 100), (5, 2, 1000)):
        _same(gi, Q, k, c, r, r1=70, expand_bits=B)
        _same(gi, Q, k, c, r, r1=9, expand_bits=B)


@pytest.mark.parametrize("H", [1, 3])
def test_queries_without_a_margin(H):
    import torch
    gi, Q = _index(20000, 64, 70, H)
    Q = Q.clone()
    Q[3] = 0.0
    Q[10] *= 1e18
    Q[11] *= 1e25
    Q[12] *= 1e-30
    _same(gi, Q, 10, 4, 100, r1=70)
    bad = Q.clone()
    bad[20, 5] = float("nan")
    bad[21, 6] = float("inf")
    bad[22, 7] = 3e38
    ids, sc = gi.search(bad, 10, 4, 100, r1=70)
    ref, rsc = gi.search(Q, 10, 4, 100, r1=70)
    keep = torch.ones(Q.shape[0], dtype=torch.bool)
    keep[20:23] = False
    assert torch.equal(ids[keep], ref[keep]) and torch.equal(sc[keep], rsc[keep])
    assert bool(((ids >= -1) & (ids < 20000)).all())


def test_large_rows_take_the_fp32_windows():
    import torch
    from paper_2205_00970_amd import lider
    X, lab, Q, _ = datagen.tiny(n=8000, d=64, ncomp=70, nq=1500, seed=75, qseed=76)
    X[17] *= 1e20
    A, b = datagen.lsh_params(4, 64, 1e20, seed=77)
    gi = lider.Index(torch.from_numpy(X).cuda(), 70, 4, 1e20, 8, (A, b),
                     assignment=torch.from_numpy(lab).cuda())
    _same(gi, torch.from_numpy(Q).cuda(), 10, 4, 100, r1=70)

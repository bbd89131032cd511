"""Small batches (up to 512 queries: layer-1 product in 16 x 16 tiles, routing
and windows in one launch, windows scored pair by pair): ids and scores equal,
bit for bit, the search with an explicit rerank shape and the same queries
inside a large batch; around the batch limit, one row to whole clusters, odd
starts, bf16, the expansion, and queries at an address no 16-byte load takes."""
import numpy as np
import pytest

from paper_2205_00970_amd import datagen

pytestmark = pytest.mark.gpu


def _index(d, kind="e2lsh", C=40):
    import torch
    from paper_2205_00970_amd import lider
    X, lab, Q, _ = datagen.tiny(n=9000, d=d, ncomp=C, nq=1200, seed=80, qseed=81)
    lab = np.where(lab == 5, 4, lab).astype(np.int32)  # an empty cluster
    A, b = datagen.lsh_params(5, d, 1.0, seed=82)
    gi = lider.Index(torch.from_numpy(X).cuda(), C, 5, 1.0, 8, (A, None if kind == "sign" else b),
                     assignment=torch.from_numpy(lab).cuda(), hash_kind=kind, storage="bf16")
    return gi, torch.from_numpy(Q).cuda()


@pytest.mark.parametrize("d,kind,B", [(64, "e2lsh", 0), (192, "e2lsh", 0), (320, "e2lsh", 0), (128, "sign", 2)])
@pytest.mark.parametrize("precision", ["f32", "bf16"])
def test_equal_to_the_large_batch(d, kind, B, precision):
    import torch
    gi, Q = _index(d, kind)
    for k, c, r, r1 in ((10, 1, 1000, 40), (1, 4, 1, 40), (17, 3, 77, 7), (100, 5, 130, 40), (10, 16, 300, 3)):
        kw = dict(r1=r1, precision=precision, expand_bits=B)
        big = gi.search(Q, k, c, r, **kw)
        for nq in (1, 3, 17, 256, 511, 512, 513):
            q = Q[:nq].contiguous()
            got = gi.search(q, k, c, r, **kw)
            ref = gi.search(q, k, c, r, tile_rows=128, pass_pairs=32, **kw)
            for a, b in ((got, ref), (got, (big[0][:nq], big[1][:nq]))):
                assert torch.equal(a[0], b[0]), (k, c, r, nq)
                assert torch.equal(a[1].view(torch.int32), b[1].view(torch.int32)), (k, c, r, nq)


def test_unaligned_queries():
    import torch
    gi, Q = _index(64)
    buf = torch.empty(50 * 64 + 1, device="cuda")
    q = buf[1:].view(50, 64)
    q.copy_(Q[:50])
    for precision in ("f32", "bf16"):
        a = gi.search(q, 10, 3, 100, r1=40, precision=precision)
        b = gi.search(Q[:50].contiguous(), 10, 3, 100, r1=40, precision=precision)
        assert torch.equal(a[0], b[0])


def test_not_finite_queries_leave_the_others():
    import torch
    gi, Q = _index(64)
    ref, rsc = gi.search(Q[:60].contiguous(), 10, 3, 100, r1=40)
    bad = Q[:60].clone()
    bad[7, 3] = float("nan")
    bad[8, 4] = float("inf")
    bad[9] *= 1e30
    ids, sc = gi.search(bad, 10, 3, 100, r1=40)
    keep = [i for i in range(60) if i not in (7, 8, 9)]
    assert torch.equal(ids[keep], ref[keep]) and torch.equal(sc[keep], rsc[keep])
    assert bool(((ids >= -1) & (ids < 9000)).all())

"""The workgroup rerank at every pass width, over rows of fewer steps than its
ring holds, of whole groups of four steps and with remainders, and over
dimensions padded to whole steps (queries in wide loads, in scalar loads, at
unaligned addresses): few and many pairs per tile.  Ids and scores equal those
of the per-wave rerank bit for bit, in fp32 and in the precision form."""
import pytest

from paper_2205_00970_amd import datagen

pytestmark = pytest.mark.gpu


def _index(d, bf16):
    import torch
    from paper_2205_00970_amd import lider
    X, lab, Q, _ = datagen.tiny(n=6000, d=d, ncomp=20, nq=900, seed=160, qseed=161)
    A, b = datagen.lsh_params(5, d, 1.0, seed=162)
    gi = lider.Index(torch.from_numpy(X).cuda(), 20, 5, 1.0, 8, (A, b), storage="bf16" if bf16 else "f32",
                     assignment=torch.from_numpy(lab).cuda())
    return gi, torch.from_numpy(Q).cuda()


def _equal(a, e):
    import torch
    assert torch.equal(a[0], e[0]) and torch.equal(a[1].view(torch.int32), e[1].view(torch.int32))


@pytest.mark.parametrize("d", [32, 64, 96, 128, 160, 224, 288, 36, 52, 100, 108, 130, 131, 300])
def test_fp32(d):
    import torch
    gi, Q = _index(d, False)
    buf = torch.empty(Q.numel() + 1, device="cuda")
    Qu = buf[1:].view_as(Q)
    Qu.copy_(Q)
    for nq, c, r in ((40, 1, 400), (200, 2, 150), (900, 4, 400)):
        e = gi.search(Q[:nq], 17, c, r, r1=20, tile_rows=64)
        for pairs in (0, 16, 32, 64, 128):
            _equal(gi.search(Q[:nq], 17, c, r, r1=20, tile_rows=128, pass_pairs=pairs), e)
        _equal(gi.search(Q[:nq], 17, c, r, r1=20), e)
        _equal(gi.search(Qu[:nq], 17, c, r, r1=20), e)


@pytest.mark.parametrize("d", [64, 128, 192, 256, 320, 448])
def test_bf16(d):
    gi, Q = _index(d, True)
    for nq, c, r in ((40, 1, 400), (200, 2, 150), (900, 4, 400)):
        e = gi.search(Q[:nq], 17, c, r, r1=20, precision="bf16", tile_rows=64)
        for pairs in (0, 16, 32, 64, 128):
            _equal(gi.search(Q[:nq], 17, c, r, r1=20, precision="bf16", tile_rows=128, pass_pairs=pairs), e)
        _equal(gi.search(Q[:nq], 17, c, r, r1=20, precision="bf16"), e)

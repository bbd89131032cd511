"""Small batches over very uneven clusters: window scores pair by pair or by
tiles, whichever the rule takes on either side of its limit (one cluster of
half the rows, whole clusters and windows of it), equal bit for bit to the
search with an explicit rerank shape."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["f32", "bf16"])
def test_equal_to_the_tiled_windows(precision):
    import torch
    from paper_2205_00970_amd import datagen, lider
    n, d, C = 400_000, 128, 200
    g = torch.Generator("cuda").manual_seed(130)
    mu = 3.0 * torch.randn(C, d, generator=g, device="cuda")
    lab = torch.randint(0, C, (n,), generator=g, device="cuda")
    lab[torch.rand(n, generator=g, device="cuda") < 0.5] = 7
    lab[lab == 11] = 12  # an empty cluster
    X = mu[lab] + 0.5 * torch.randn(n, d, generator=g, device="cuda")
    Q = X[torch.randint(0, n, (60,), generator=g, device="cuda")] + 0.05 * torch.randn(60, d, generator=g, device="cuda")
    A, b = datagen.lsh_params(6, d, 2.0, seed=131)
    gi = lider.Index(X, C, 6, 2.0, 16, (A, b), assignment=lab.int(), storage="bf16" if precision == "bf16" else "f32")
    for nq, c in ((1, 1), (2, 1), (12, 1), (50, 1), (12, 4)):
        for r in (64, 5000, int(gi.max_cluster)):
            a = gi.search(Q[:nq], 10, c, r, r1=C, precision=precision)
            e = gi.search(Q[:nq], 10, c, r, r1=C, precision=precision, tile_rows=128)
            assert torch.equal(a[0], e[0]) and torch.equal(a[1].view(torch.int32), e[1].view(torch.int32)), (nq, c, r)

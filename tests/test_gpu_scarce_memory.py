"""An index loaded where device memory holds what it needs but not its optional
operand-ordered fp32 copy as well: the load succeeds, and the search returns
what it returns with room for the copy."""
import os

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [100])
def test_load_without_room_for_the_optional_copy(tmp_path, d):
    import torch
    from paper_2205_00970_amd import datagen, lider
    n, C = 2_000_000, 400
    g = torch.Generator("cuda").manual_seed(140)
    X = torch.randn(n, d, generator=g, device="cuda")
    Q = X[:50] + 0.1 * torch.randn(50, d, generator=g, device="cuda")
    lab = (torch.arange(n, device="cuda") % C).int()
    A, b = datagen.lsh_params(4, d, 2.0, seed=141)
    gi = lider.Index(X, C, 4, 2.0, 8, (A, b), assignment=lab, storage="bf16")
    ids, sc = gi.search(Q, 10, 2, 500, r1=C)
    path = os.path.join(tmp_path, "index")
    gi.save(path)
    gi.close()
    del X, lab
    torch.cuda.empty_cache()
    # the rows and their bf16 copy (1.2 GB), what an index keeps beside them
    # (0.2 GB), and most of the fp32 copy (1.0 GB)
    room = 2_150_000_000
    free = torch.cuda.mem_get_info()[0]
    fill = torch.empty(free - room, dtype=torch.uint8, device="cuda")
    try:
        gl = lider.Index.load(path)
        ids2, sc2 = gl.search(Q, 10, 2, 500, r1=C)
        assert torch.equal(ids, ids2)
        assert torch.equal(sc, sc2)
        gl.close()
    finally:
        del fill
        torch.cuda.empty_cache()

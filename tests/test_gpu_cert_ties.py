"""Certified lists with more exactly equal scores than the selection's tie
table holds, in a chunk merged with the best so far: a zero query (every
candidate listed, every score 0) and a group of identical rows, for the
1,024-thread and the 256-thread rerank.  The tied places go to the smallest
ids, as in the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2205_00970_amd import datagen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq", [40, 1100])
@pytest.mark.parametrize("k", [65, 100, 128])
def test_tied_places_go_to_the_smallest_ids(nq, k):
    import torch
    from paper_2205_00970_amd import lider
    n, C, d = 36000, 12, 64
    X, lab, Q, _ = datagen.tiny(n=n, d=d, ncomp=C, nq=nq, seed=94, qseed=95)
    at = np.nonzero(lab == 2)[0][:2500]
    assert at.size == 2500
    X[at] = 2.0 * X[at[0]]  # ahead of every other row for their own direction
    Q[0] = 0.0
    Q[1] = X[at[0]]
    Q[2] = 0.5 * X[at[0]]
    A, b = datagen.lsh_params(5, d, 1.0, seed=96)
    gi = lider.Index(torch.from_numpy(X).cuda(), C, 5, 1.0, 8, (A, b), storage="bf16",
                     assignment=torch.from_numpy(lab).cuda())
    oi = oracle.Index(X, C, A, b, 5, 1.0, 8, assignment=lab)
    Qd = torch.from_numpy(Q).cuda()
    for c, r in ((1, 5000), (4, 5000), (4, 2500)):
        ids, sc = gi.search(Qd, k, c, r, r1=C, precision="bf16")
        oids, osc = oi.search(Q[:3], k, c, r, C)
        assert np.array_equal(ids[:3].cpu().numpy(), oids)
        assert np.allclose(sc[:3].cpu().numpy(), osc, rtol=1e-5, atol=0)

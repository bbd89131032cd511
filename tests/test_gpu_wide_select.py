"""The workgroup selection (k <= 128) and the ranking of certified lists:
every register count (2,048 to 32,768 candidates), the radix forms past their
limits, exact ties at the boundary and past the list's room, several arrays,
fewer candidates than k, against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2205_00970_amd import datagen

from parity_util import compare_topk

pytestmark = pytest.mark.gpu


def _pair(H=1, copies=0, n=24000, C=12, d=32):
    import torch
    from paper_2205_00970_amd import lider
    X, lab, Q, _ = datagen.tiny(n=n, d=d, ncomp=C, nq=1100, seed=90, qseed=91)
    if copies:
        at = np.nonzero(lab == 2)[0][:copies]
        X[at] = X[at[0]]
        Q[:30] = X[at[0]]
    A, b = datagen.lsh_params(5, d, 1.0, seed=92, n_arrays=H)
    gi = lider.Index(torch.from_numpy(X).cuda(), C, 5, 1.0, 8, (A, b), n_arrays=H, storage="bf16",
                     assignment=torch.from_numpy(lab).cuda())
    oi = oracle.Index(X, C, A, b, 5, 1.0, 8, assignment=lab, n_arrays=H)
    return X, Q, gi, oi


@pytest.mark.parametrize("H,copies", [(1, 0), (1, 120), (1, 900), (3, 0), (2, 900)])
@pytest.mark.parametrize("precision", ["f32", "bf16"])
def test_top_k_equals_the_oracle(H, copies, precision):
    import torch
    X, Q, gi, oi = _pair(H, copies)
    for nq in (40, 1100):
        Qd = torch.from_numpy(Q[:nq]).cuda()
        for k, c, r in ((100, 1, 1000), (65, 1, 60), (128, 4, 500), (100, 4, 1000), (127, 8, 1000),
                        (100, 12, 1300), (100, 12, 5000), (17, 4, 1000), (64, 8, 1000),
                        (33, 12, 1300)):
            ids, sc = gi.search(Qd, k, c, r, r1=12, precision=precision)
            oids, osc = oi.search(Q[:nq], k, c, r, 12)
            compare_topk(X, Q[:nq], ids.cpu().numpy(), sc.cpu().numpy(), oids, osc)


@pytest.mark.parametrize("precision", ["f32", "bf16"])
def test_past_the_workgroup_limit_equals_the_oracle(precision):
    import torch
    X, Q, gi, oi = _pair(n=44000)
    Qd = torch.from_numpy(Q[:50]).cuda()
    for k, c, r in ((100, 8, 3700), (100, 12, 5000), (64, 8, 3700), (40, 12, 5000)):
        ids, sc = gi.search(Qd, k, c, r, r1=12, precision=precision)
        oids, osc = oi.search(Q[:50], k, c, r, 12)
        compare_topk(X, Q[:50], ids.cpu().numpy(), sc.cpu().numpy(), oids, osc)

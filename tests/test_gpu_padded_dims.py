"""Dimensions that are not multiples of 32: the operand-ordered copy padded with
zeros, the workgroup and pair reranks on it and the split layer-1 product,
against the FP64 oracle and, bit for bit, the row-major rerank."""
import numpy as np
import pytest

import oracle
from paper_2205_00970_amd import datagen

from parity_util import compare_debug, compare_topk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [20, 33, 44, 50, 95, 100, 131, 300])
def test_search_equals_the_oracle(d):
    import torch
    from paper_2205_00970_amd import lider
    X, lab, Q, _ = datagen.tiny(n=7000, d=d, ncomp=20, nq=900, seed=95, qseed=96)
    A, b = datagen.lsh_params(5, d, 1.0, seed=97)
    gi = lider.Index(torch.from_numpy(X).cuda(), 20, 5, 1.0, 8, (A, b),
                     assignment=torch.from_numpy(lab).cuda())
    oi = oracle.Index(X, 20, A, b, 5, 1.0, 8, assignment=lab)
    buf = torch.empty(900 * d + 1, device="cuda")  # rows at addresses of 4 bytes only
    odd = buf[1:].view(900, d)
    odd.copy_(torch.from_numpy(Q))
    for nq in (5, 900):
        for Qd in (torch.from_numpy(Q[:nq]).cuda(), odd[:nq]):
            for k, c, r, r1 in ((10, 3, 100, 20), (17, 2, 1000, 7), (10, 1, 400, 20)):
                ids, sc, dbg = gi.search(Qd, k, c, r, r1=r1, debug=True)
                oids, osc, odbg = oi.search(Q[:nq], k, c, r, r1, debug=True)
                compare_debug(dbg, odbg)
                compare_topk(X, Q[:nq], ids.cpu().numpy(), sc.cpu().numpy(), oids, osc)
                ref = gi.search(Qd, k, c, r, r1=r1, tile_rows=64)
                assert torch.equal(ids, ref[0]) and torch.equal(sc, ref[1])

"""The dist_e expansion decided 256 positions per step: the merge rule on the
CPU, and windows around the step's size against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2205_00970_amd import datagen

from parity_util import compare_debug


def test_heads_merge_like_running_maxima():
    """Taking the smaller head (ties left) of two sequences in any order takes
    as many from the left as the count over l of A_l <= B_{T-1-l}, A and B the
    running maxima; exhausted sides never win."""
    g = np.random.default_rng(0)
    far = np.iinfo(np.int32).max
    for _ in range(3000):
        a = g.integers(0, 6, g.integers(0, 9)).tolist()
        b = g.integers(0, 6, g.integers(0, 9)).tolist()
        for T in range(len(a) + len(b) + 1):
            i = j = 0
            for _ in range(T):
                if i < len(a) and (j == len(b) or a[i] <= b[j]):
                    i += 1
                else:
                    j += 1
            A = np.maximum.accumulate(a + [far] * (T + 1 - min(T, len(a))))
            B = np.maximum.accumulate(b + [far] * (T + 1 - min(T, len(b))))
            assert i == sum(A[x] <= B[T - 1 - x] for x in range(T)), (a, b, T)


@pytest.mark.gpu
@pytest.mark.parametrize("m,B", [(10, 3), (16, 16)])
def test_windows_around_a_step(m, B):
    import torch
    from paper_2205_00970_amd import lider
    X, lab, Q, _ = datagen.tiny(n=6000, d=64, ncomp=4, nq=64, seed=61, qseed=62)
    X, Q = datagen.normalize_rows(X), datagen.normalize_rows(Q)
    lab = np.where(lab == 0, np.arange(6000) % 2 * 4, lab).astype(np.int32)  # 5 clusters, 750-1500 rows
    A, _ = datagen.lsh_params(m, 64, 1.0, seed=63)
    gi = lider.Index(torch.from_numpy(X).cuda(), 5, m, 1.0, 8, (A, None),
                     assignment=torch.from_numpy(lab).cuda(), hash_kind="sign")
    oi = oracle.Index(X, 5, A, np.zeros(2 * m, np.float32), m, 1.0, 8, assignment=lab,
                      hash_kind="sign")
    Qd = torch.from_numpy(Q).cuda()
    for r in (2, 3, 255, 256, 257, 258, 513, 514, 769, 1400, 1600):
        _, _, dbg = gi.search(Qd, 10, 3, r, r1=3, debug=True, expand_bits=B)
        _, _, odbg = oi.search(Q, 10, 3, r, 3, debug=True, expand_bits=B)
        compare_debug(dbg, odbg)

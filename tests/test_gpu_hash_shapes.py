"""Query and corpus hashing at the edges of its workgroup forms (one, two, four
and sixteen waves), of its 16-dimension steps and of its 32-hash blocks, with
rows at 16-byte and at 4-byte addresses, against the FP64 oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("n,d,nh", [
    (1, 1, 1), (17, 15, 4), (700, 16, 17), (700, 31, 33), (5105, 64, 4), (5088, 64, 16), (2040, 64, 5),
    (2048, 65, 32), (3201, 100, 8), (9000, 100, 16), (6400, 130, 16), (1000, 300, 40), (9601, 300, 16),
    (100, 512, 16), (100, 768, 33), (30, 777, 8), (1, 1024, 16)])
def test_digits_equal_the_oracle(n, d, nh, offset):
    import torch
    from paper_2205_00970_amd import lider
    rng = np.random.default_rng(n + 7 * d + nh)
    X = rng.standard_normal((n, d)).astype(np.float32)
    A = rng.standard_normal((nh, d)).astype(np.float32)
    b = rng.uniform(0.0, 2.0, nh).astype(np.float32)
    room = torch.empty(n * d + offset, device="cuda")
    Xd = room[offset:].view(n, d)
    Xd.copy_(torch.from_numpy(X))
    got = lider.hash(Xd, torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda(), 2.0)
    assert np.array_equal(got.cpu().numpy(), oracle.digits(X, A, b, 2.0))

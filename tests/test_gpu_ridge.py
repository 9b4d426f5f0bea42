"""The ridge solve's divisions by reciprocal and their limits, and one to seventeen blocks of 16 rows: penalties and data at the
ends of the range, where the quotients are divided, zeros, infinities.  To the bit as the oracle, whose operations it repeats."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


# (C, scale of the data, penalty, what is in the first rows)
@pytest.mark.parametrize("case", [(1, 1.0, 1.0, "zeros"), (2, 1.0, 1e-300, ""), (3, 1e-38, 1e200, ""), (3, 1e-44, 1.0, ""), (4, 1e37, 1e-3, "zeros"),
                                  (5, 1e37, 1e300, ""), (3, 1.0, 1.0, "inf"), (17, 1.0, 0.37, "zeros"), (16, 3e-3, 1e-2, "")], ids=str)
def test_prototypes_to_the_bit(case):
    import torch
    import paper_2106_10860_amd as mad
    C, scale, lam, kind = case
    print("case", case, flush=True)
    rng = np.random.default_rng(int(C * 1000))
    N, D = 150 + 7 * C, 2 * C + 5
    A = (rng.standard_normal((N, D)) * scale).astype(np.float32)
    if kind == "zeros":
        A[:, :3] = 0.0
        A[: N // 2] = 0.0
    if kind == "inf":
        A[3, 1], A[5, 2] = np.inf, -np.inf
    codes = np.minimum(rng.integers(0, 18, size=(N, C)), 14).astype(np.uint8)       # one code of every codebook is not used
    want = oracle.ridge_prototypes(codes, A, lam).astype(np.float32)
    bounds = [(2 * c, 2 * c + 2) for c in range(C)]
    got = mad.maddness_learn_prototypes(torch.from_numpy(codes).cuda(), torch.from_numpy(A).cuda(), bounds, ridge=True, lam=lam)
    torch.cuda.synchronize()
    got = got.cpu().numpy().reshape(want.shape)
    assert np.array_equal(got, want, equal_nan=True), (np.argwhere(got != want)[:5], got[got != want][:5], want[got != want][:5])

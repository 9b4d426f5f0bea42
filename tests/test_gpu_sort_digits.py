"""The learner's sort looks only at the bits in which a column's values differ: columns of one to four digits side by side,
constant ones, negative ones, widths whose threads see one column in all turns and widths whose do not, one launch for all
digits and two launches a digit.  Trees equal the oracle's."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,widths", [(512, [8, 3]), (513, [8, 16]), (700, [7, 8, 3]), (8192, [16, 5]), (8193, [6, 8]), (9001, [48]), (12000, [20, 4])], ids=str)
def test_trees_of_columns_with_few_bits(N, widths):
    import torch
    import paper_2106_10860_amd as mad
    print("case", N, widths, flush=True)
    rng = np.random.default_rng(N)
    D = sum(widths)
    A = np.empty((N, D), np.float32)
    for j in range(D):
        bits = [1, 3, 7, 9, 12, 16, 22, 24][j % 8]                # of a whole number; the last ones fill a mantissa
        v = rng.integers(0, 1 << bits, size=N).astype(np.float64) * 2.0 ** rng.integers(-20, 20)
        if j % 5 == 1: v = -v
        if j % 5 == 2: v = v - v.mean().round()
        if j % 7 == 3: v = rng.standard_normal(N)                 # any bits
        if j % 11 == 4: v = np.full(N, -3.5)
        A[:, j] = v
    A[0] = A[N // 2]                                              # (the first row is nothing special)
    at = np.concatenate([[0], np.cumsum(widths)])
    subspaces = [(int(at[c]), int(at[c + 1])) for c in range(len(widths))]
    sd, th, codes = mad.maddness_learn_trees(torch.from_numpy(A).cuda(), subspaces)
    torch.cuda.synchronize()
    want_sd, want_th, want_codes, _ = oracle.learn_trees(A, subspaces)
    assert (sd.cpu().numpy() == want_sd).all() and (th.cpu().numpy() == want_th).all()
    assert (codes.cpu().numpy() == want_codes).all()

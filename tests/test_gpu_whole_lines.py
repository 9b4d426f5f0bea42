"""Outputs whose rows begin inside 128-byte lines and take several wavefronts' columns: every result where it belongs,
equal to the oracle's to the bit, and nothing written beside the rows.  Split columns larger than the last-level cache, which are
read past it: the codes of the general kernel."""
import numpy as np
import pytest

import oracle
from test_gpu_tables_and_few_rows import dev, problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mad():
    import torch
    import paper_2106_10860_amd as m
    assert torch.cuda.is_available()
    m.lib()
    return m


# (N, M, C, floats between rows, floats the output starts after a line, whole lines or another kernel): rows of a class that make
# a whole number of groups of 16 and that do not, 2 to 32 classes, one to many blocks of columns, blocks that end with the row and
# that go on with the next one's columns (on a multiple of four and not), the last row's last line, padding codebooks; padding,
# other alignments, few results and shapes that other kernels write as fast
CUT = [
    (16384, 1000, 32, 0, 0, True), (16390, 1000, 32, 0, 0, True), (49001, 257, 32, 0, 0, True), (28100, 449, 30, 0, 0, True),
    (53007, 252, 30, 0, 0, True), (28001, 450, 16, 0, 0, True), (18700, 676, 8, 0, 0, True), (18697, 673, 31, 0, 0, True),
    (65201, 193, 64, 0, 0, True), (95001, 290, 40, 0, 0, True), (89900, 141, 50, 0, 0, True), (96800, 130, 33, 0, 0, True),
    (193600, 65, 32, 0, 0, True), (93000, 136, 64, 0, 0, True), (99079, 127, 5, 0, 0, True), (29001, 1022, 64, 0, 0, True),
    (92003, 144, 24, 0, 0, True), (36001, 368, 32, 0, 0, True), (70000, 188, 16, 0, 0, True), (48001, 272, 16, 0, 0, True),
    (43400, 290, 40, 0, 0, False), (16386, 1022, 64, 0, 0, False), (36001, 368, 8, 0, 0, False), (139000, 188, 16, 0, 0, False),
    (79001, 170, 30, 0, 0, False), (78001, 162, 48, 0, 0, False), (101001, 125, 31, 0, 0, False),
    (16385, 452, 24, 4, 0, False), (16384, 1000, 32, 1, 0, False), (16390, 1000, 32, 0, 4, False), (33, 514, 64, 0, 0, False),
    (16384, 449, 30, 0, 1, False), (52000, 250, 30, 0, 0, False),
]


@pytest.mark.parametrize("shape", CUT, ids=lambda s: "N%d_M%d_C%d_pad%d_at%d" % s[:5])
def test_scan_writes_whole_lines(mad, shape, blocks):
    import torch
    N, M, C, pad, at, lines = shape
    print("case", shape, flush=True)
    _, _, _, luts, scale, offset = problem(N + M, 8, 4 * C, M, C)
    rng = np.random.default_rng(M)
    codes = rng.integers(0, 256, size=(N, (C + 1) // 2)).astype(np.uint8)
    if C % 2:
        codes[:, -1] &= 15
    want_out, _, _ = oracle.scan(codes, C, luts, scale, offset)
    ldo = M + pad
    raw = torch.full((at + N * ldo + 64,), -7.0, dtype=torch.float32, device="cuda")
    out = raw[at:at + N * ldo].reshape(N, ldo)[:, :M]
    mad.maddness_scan(C, dev(codes), dev(luts), dev(scale), dev(offset), out=out)
    kernel = mad.maddness_last_kernel()
    torch.cuda.synchronize()
    assert kernel.startswith("mfma_scan_kernel") and ("whole lines" in kernel) == lines or (
        blocks and not lines and kernel.startswith("fused_blocks_kernel, scan")), kernel
    assert (out.cpu().numpy() == want_out).all()
    got = raw.cpu().numpy()
    assert (got[:at] == -7).all() and (got[at + (N - 1) * ldo + M:] == -7).all()
    assert (got[at:at + N * ldo].reshape(N, ldo)[:, M:][:-1] == -7).all()


@pytest.mark.parametrize("M, C", [(20001, 8), (9002, 33)], ids=str)
def test_scan_whole_lines_of_very_wide_rows(mad, M, C):
    """Rows with more blocks of columns than a class of them has workgroups in a turn of the chip, against the general kernel."""
    import torch
    N = 16390
    print("case wide", N, M, C, flush=True)
    _, _, _, luts, scale, offset = problem(M, 8, 4 * C, M, C)
    codes = torch.randint(0, 256, (N, (C + 1) // 2), generator=torch.Generator(device="cuda").manual_seed(M), device="cuda", dtype=torch.int32).to(torch.uint8)
    if C % 2:
        codes[:, -1] &= 15
    args = (C, codes, dev(luts), dev(scale), dev(offset))
    got, _ = mad.maddness_scan(*args)
    assert mad.maddness_last_kernel().startswith("mfma_scan_kernel, whole lines"), mad.maddness_last_kernel()
    try:
        mad.maddness_set_option(mad.MADDNESS_OPT_KERNELS, mad.MADDNESS_KERNELS_GENERAL)
        want, _ = mad.maddness_scan(*args)
        assert mad.maddness_last_kernel().startswith("scan_kernel"), mad.maddness_last_kernel()
    finally:
        mad.maddness_set_option(mad.MADDNESS_OPT_KERNELS, 0)
    torch.cuda.synchronize()
    assert torch.equal(got, want)


# once: every column is split once; twice: one is split again on another level of its codebook or in another codebook; few: fewer
# columns than splits
@pytest.mark.parametrize("dtype, N, C, splits", [("float32", (1 << 20) + 3, 16, "once"), ("float16", (1 << 19) + 6, 64, "once"),
                                                 ("bfloat16", (1 << 20) + 5, 32, "once"), ("float16", (1 << 19) + 6, 64, "twice"),
                                                 ("float32", (1 << 20) + 3, 16, "twice"), ("bfloat16", (1 << 20) + 5, 32, "few")])
def test_encode_columns_larger_than_the_caches(mad, dtype, N, C, splits):
    import torch
    print("case columns", dtype, N, C, splits, flush=True)
    D = 4 * C - (splits == "few")
    g = torch.Generator(device="cuda").manual_seed(C)
    pitch = (N + 3) // 4 * 4
    A = torch.randn((D, pitch), generator=g, device="cuda").clamp_(min=0).to(getattr(torch, dtype))[:, :N]
    rng = np.random.default_rng(C)
    sd = np.stack([rng.permutation(4) + 4 * c for c in range(C)]).astype(np.int32)
    if splits == "twice":
        sd[-1, 3] = sd[-1, 0] if C == 16 else sd[0, 1]
    sd = np.minimum(sd, D - 1)
    th = np.abs(rng.standard_normal((C, 16))).astype(np.float32)
    params = mad.Params(dev(sd), dev(th))
    got = mad.maddness_encode_typed(params, A, col_major=True)
    kernel = mad.maddness_last_kernel()
    torch.cuda.synchronize()
    assert kernel.startswith("cols_kernel") and ("NT = true" in kernel) == (splits != "few"), kernel
    # a walk of the same trees on the same values
    node = torch.zeros((N, C), dtype=torch.int64, device="cuda")
    at, thd, sdd = torch.arange(C, device="cuda"), dev(th), dev(sd).long()
    for t in range(4):
        node = 2 * node + (A[sdd[:, t]].t().float() >= thd[at, (1 << t) - 1 + node]).long()
    want = (node[:, 0::2] | (node[:, 1::2] << 4)).to(torch.uint8)
    assert torch.equal(got, want)

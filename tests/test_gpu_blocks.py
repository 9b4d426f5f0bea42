"""The fused kernel that works by blocks of rows and columns: every kernel size, one to sixteen tiles of columns to a
block, one chunk of rows to a workgroup and several (one or two workgroups to a compute unit), tables beside the staged
rows and in their place, tables whose last pieces run over their end, rows on any element.  The reference is the
oracle's scalar statement for few rows; for many, the library's general kernels, which the other tests hold against it.
Sums are whole numbers and one rounding follows: everything is equal to the bit."""
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


# (N, D, M, C, dtype, elements between rows, elements before the first, bytes before the tables)
CASES = [
    # one row, and fewer than a group of 16
    (1, 64, 128, 16, "f32", 0, 0, 0), (1, 27, 1, 4, "u8", 0, 1, 0), (2, 1024, 512, 64, "f16", 0, 0, 0), (7, 333, 300, 30, "bf16", 1, 0, 3), (15, 61, 33, 7, "f32", 0, 1, 0),
    # fewest rows; one column; a table of 16 bytes to a codebook, of which the last piece is all there is
    (16, 64, 1, 32, "f32", 0, 0, 0), (17, 33, 129, 16, "f32", 0, 1, 1), (31, 48, 15, 48, "f32", 0, 0, 3),
    # kernel sizes with and without codebooks that do not exist
    (700, 27, 200, 4, "f32", 0, 0, 0), (515, 61, 100, 7, "f32", 3, 0, 2), (333, 250, 255, 15, "f16", 1, 3, 0),
    (300, 96, 77, 21, "u8", 0, 5, 1), (257, 333, 64, 31, "bf16", 0, 0, 0), (130, 240, 48, 43, "f32", 0, 3, 0),
    (90, 505, 127, 63, "f32", 7, 0, 5), (64, 1024, 130, 64, "u8", 0, 0, 0),
    # kernel sizes of which up to half is padding
    (300, 27, 40, 1, "f32", 0, 0, 0), (333, 45, 130, 5, "f16", 1, 0, 1), (257, 99, 17, 9, "u8", 0, 3, 0), (130, 170, 255, 17, "f32", 0, 1, 3),
    (90, 250, 31, 25, "bf16", 3, 0, 0), (70, 333, 100, 33, "f32", 0, 0, 5), (65, 505, 129, 49, "u8", 0, 5, 2), (40001, 99, 90, 11, "f16", 0, 0, 0),
    # blocks of one to eight tiles, and more than one block of columns, the last one with a column
    (1000, 128, 16, 32, "f32", 0, 0, 0), (1000, 128, 32, 32, "f32", 0, 0, 0), (1000, 128, 60, 32, "f32", 0, 0, 0),
    (400, 512, 257, 32, "f32", 0, 0, 0), (200, 64, 1025, 24, "f32", 0, 0, 4),
    # rows of 4 to 8 KiB on any element; rows of 8 KiB; tables in the place of the first rows
    (300, 1025, 40, 64, "f32", 0, 1, 0), (40, 2047, 130, 48, "f32", 1, 3, 1), (4000, 1501, 17, 16, "f32", 2, 1, 0),
    (40, 2048, 96, 64, "f32", 0, 0, 0), (9000, 512, 512, 32, "bf16", 0, 0, 0), (4100, 1024, 128, 64, "f32", 0, 0, 0),
    # several chunks to a workgroup: wide blocks; two workgroups to a compute unit; the last chunk with a row
    (3001, 384, 1000, 24, "f32", 0, 0, 0), (40001, 120, 90, 15, "f32", 0, 0, 0), (131077, 27, 20, 4, "f32", 0, 0, 0),
    (65537, 64, 300, 8, "f16", 0, 0, 0), (33000, 480, 16, 30, "f32", 0, 2, 0), (50000, 528, 7, 48, "f32", 0, 0, 0),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "N%d_D%d_M%d_C%d_%s_p%d_o%d_t%d" % c)
def test_blocks_of_rows_and_columns(mad, case):
    import torch
    N, D, M, C, dtype, pad, before, at = case
    print("case", case, flush=True)
    A, sd, th, luts, scale, offset = problem(N + D + M, min(N, 2048), D, M, C)
    kind = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "u8": torch.uint8}[dtype]
    full = torch.full((before + N * (D + pad),), 1, dtype=kind, device="cuda")
    A_d = full[before:].view(N, D + pad)[:, :D]
    values = (dev(A) * (60 if dtype == "u8" else 1)).clamp(max=255).to(kind)
    A_d.copy_(values[torch.arange(N, device="cuda") % len(A)])
    raw = torch.zeros(luts.size + at, dtype=torch.uint8, device="cuda")
    raw[at:] = dev(luts).reshape(-1)
    luts_d = raw[at:].reshape(C, 16, M)
    params = mad.Params(dev(sd), dev(th))

    def run():
        acc = torch.zeros((N, M), dtype=torch.int16, device="cuda")
        codes = torch.zeros((N, (C + 1) // 2), dtype=torch.uint8, device="cuda")
        out = mad.maddness_encode_scan_typed(params, A_d, luts_d, dev(scale), dev(offset), acc=acc, codes=codes)
        return out, acc, codes, mad.maddness_last_kernel()

    out, acc, codes, kernel = run()
    torch.cuda.synchronize()
    assert kernel.startswith("fused_blocks_kernel, A by rows"), kernel
    if N <= 2048:
        want_out, want_acc, want_codes = oracle.encode_scan(A_d.float().cpu().numpy().copy(), sd, th, luts, scale, offset)
        assert (codes.cpu().numpy() == want_codes).all()
        assert (acc.cpu().numpy().view(np.uint16) == want_acc).all()
        assert (out.cpu().numpy() == want_out).all()
    else:
        mad.maddness_set_option(mad.MADDNESS_OPT_KERNELS, mad.MADDNESS_KERNELS_GENERAL)
        try:
            want_out, want_acc, want_codes, general = run()
        finally:
            mad.maddness_set_option(mad.MADDNESS_OPT_KERNELS, mad.MADDNESS_KERNELS_AUTO)
        torch.cuda.synchronize()
        assert general.startswith("scan_kernel"), general
        assert torch.equal(codes, want_codes) and torch.equal(acc, want_acc) and torch.equal(out, want_out)
    # results alone, into rows with columns between them that stay as they are
    wide = torch.full((N, M + 5), -7.0, device="cuda")
    mad.maddness_encode_scan_typed(params, A_d, luts_d, dev(scale), dev(offset), out=wide[:, :M])
    assert mad.maddness_last_kernel() == kernel
    torch.cuda.synchronize()
    assert torch.equal(wide[:, :M], out) and bool((wide[:, M:] == -7.0).all())


# (N, D, M, C, dtype, elements between columns): less than a run of 64 rows, whole runs, a row more, several runs to a workgroup
# and workgroups without any; kernel sizes with and without codebooks that do not exist; one to eight tiles of columns
COLUMNS = [
    (1, 64, 128, 16, "f32", 0), (2, 300, 130, 64, "f16", 1), (7, 30, 33, 9, "u8", 0), (15, 200, 1000, 48, "bf16", 3),
    (16, 64, 1, 16, "f32", 0), (63, 300, 130, 64, "f16", 1), (64, 27, 64, 4, "u8", 3), (65, 200, 1000, 48, "f32", 0),
    (577, 61, 35, 7, "bf16", 0), (1025, 128, 255, 15, "f32", 2), (2049, 256, 512, 32, "u8", 0), (4100, 96, 129, 21, "f16", 5),
    (700, 27, 40, 1, "f32", 0), (333, 45, 130, 5, "f16", 1), (1025, 99, 17, 9, "u8", 0), (130, 170, 255, 17, "f32", 3), (2000, 250, 31, 25, "bf16", 0),
    (90, 333, 100, 33, "f32", 0), (577, 505, 129, 49, "u8", 1),
    (9001, 240, 100, 31, "f32", 1), (70001, 72, 20, 8, "u8", 0), (70001, 128, 100, 16, "bf16", 7), (40000, 330, 90, 63, "f32", 0),
]


@pytest.mark.parametrize("case", COLUMNS, ids=lambda c: "N%d_D%d_M%d_C%d_%s_p%d" % c)
def test_blocks_of_a_stored_by_columns(mad, case):
    import torch
    N, D, M, C, dtype, pad = case
    print("case", case, flush=True)
    A, sd, th, luts, scale, offset = problem(N + D + M, min(N, 2049), D, M, C)
    kind = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "u8": torch.uint8}[dtype]
    values = (dev(A) * (60 if dtype == "u8" else 1)).clamp(max=255).to(kind)
    full = torch.zeros((D, N + pad), dtype=kind, device="cuda")
    full[:, :N] = values[torch.arange(N, device="cuda") % len(A)].t()
    A_d = full[:, :N]
    params = mad.Params(dev(sd), dev(th))

    def run():
        acc = torch.zeros((N, M), dtype=torch.int16, device="cuda")
        codes = torch.zeros((N, (C + 1) // 2), dtype=torch.uint8, device="cuda")
        out = mad.maddness_encode_scan_typed(params, A_d, dev(luts), dev(scale), dev(offset), col_major=True, acc=acc, codes=codes)
        return out, acc, codes, mad.maddness_last_kernel()

    out, acc, codes, kernel = run()
    torch.cuda.synchronize()
    assert kernel.startswith("fused_blocks_kernel, A by columns"), kernel
    if N <= 2049:
        want_out, want_acc, want_codes = oracle.encode_scan(A_d.float().t().cpu().numpy().copy(), sd, th, luts, scale, offset)
        assert (codes.cpu().numpy() == want_codes).all()
        assert (acc.cpu().numpy().view(np.uint16) == want_acc).all()
        assert (out.cpu().numpy() == want_out).all()
    else:
        mad.maddness_set_option(mad.MADDNESS_OPT_KERNELS, mad.MADDNESS_KERNELS_GENERAL)
        try:
            want_out, want_acc, want_codes, general = run()
        finally:
            mad.maddness_set_option(mad.MADDNESS_OPT_KERNELS, mad.MADDNESS_KERNELS_AUTO)
        torch.cuda.synchronize()
        assert general.startswith("scan_kernel"), general
        assert torch.equal(codes, want_codes) and torch.equal(acc, want_acc) and torch.equal(out, want_out)


# (N, D, M, C, elements between rows, before the first, bytes before the tables): two to eight tiles of columns, the end of the
# tables, rows on any element, one chunk to a workgroup and several
AVERAGES = [
    (1, 64, 128, 16, 0, 0, 0), (2, 512, 31, 64, 0, 1, 0), (15, 100, 300, 32, 1, 0, 1),
    (16, 64, 1, 16, 0, 0, 0), (33, 100, 31, 64, 0, 1, 3), (700, 512, 100, 32, 0, 0, 0), (300, 64, 1000, 48, 4, 0, 1),
    (1025, 333, 129, 32, 1, 0, 0), (2048, 1024, 130, 64, 0, 0, 0), (4100, 128, 257, 16, 0, 3, 2), (20001, 256, 60, 32, 0, 0, 0),
    (9845, 1024, 128, 64, 0, 0, 0), (30000, 64, 300, 16, 0, 0, 0), (65536, 2048, 130, 32, 0, 0, 0), (20000, 2040, 900, 32, 0, 0, 0),
]
# more turns of long rows, which the general kernel takes faster
AVERAGES_LEFT = [(65537, 2048, 130, 32, 0, 0, 0), (27000, 2040, 900, 32, 0, 0, 0)]


@pytest.mark.parametrize("case", AVERAGES + AVERAGES_LEFT, ids=lambda c: "N%d_D%d_M%d_C%d_p%d_o%d_t%d" % c)
def test_averages_by_blocks(mad, case):
    import torch
    N, D, M, C, pad, before, at = case
    print("case", case, flush=True)
    A, sd, th, luts, scale, offset = problem(N + D + M, min(N, 2048), D, M, C)
    full = torch.full((before + N * (D + pad),), 1.0, device="cuda")
    A_d = full[before:].view(N, D + pad)[:, :D]
    A_d.copy_(dev(A)[torch.arange(N, device="cuda") % len(A)])
    raw = torch.zeros(luts.size + at, dtype=torch.uint8, device="cuda")
    raw[at:] = dev(luts).reshape(-1)
    luts_d = raw[at:].reshape(C, 16, M)
    params = mad.Params(dev(sd), dev(th))

    def run():
        acc = torch.zeros((N, M), dtype=torch.int16, device="cuda")
        codes = torch.zeros((N, C // 2), dtype=torch.uint8, device="cuda")
        out = mad.maddness_encode_scan_averaged(params, A_d, luts_d, dev(scale), dev(offset), acc=acc, codes=codes)
        return out, acc, codes, mad.maddness_last_kernel()

    out, acc, codes, kernel = run()
    torch.cuda.synchronize()
    assert kernel.startswith("fused_blocks_kernel, averages") == (case not in AVERAGES_LEFT), kernel
    if N <= 2048:
        want_codes = oracle.encode_scan(A_d.cpu().numpy().copy(), sd, th, luts, scale, offset)[2]
        want_out, want_acc = oracle.scan_averaged(want_codes, C, luts, scale, offset)
        assert (codes.cpu().numpy() == want_codes).all()
        assert (acc.cpu().numpy().view(np.uint16) == want_acc).all()
        assert (out.cpu().numpy() == want_out).all()
    else:
        mad.maddness_set_option(mad.MADDNESS_OPT_KERNELS, mad.MADDNESS_KERNELS_GENERAL)
        try:
            want_out, want_acc, want_codes, general = run()
        finally:
            mad.maddness_set_option(mad.MADDNESS_OPT_KERNELS, mad.MADDNESS_KERNELS_AUTO)
        torch.cuda.synchronize()
        assert general.startswith("scan_kernel"), general
        assert torch.equal(codes, want_codes) and torch.equal(acc, want_acc) and torch.equal(out, want_out)


# (N, M, C, floats between rows, bytes before the codes, bytes before the tables): fewest rows, one column, every kernel size with and
# without codebooks that do not exist, codes by eight, four and single bytes, one block of columns and several, one chunk and several
SCANS = [
    (1, 1, 4, 0, 0, 0), (1, 300, 64, 0, 0, 0), (2, 129, 7, 1, 1, 0), (15, 100, 32, 0, 0, 3),
    (16, 1, 4, 0, 0, 0), (17, 300, 64, 0, 0, 0), (33, 64, 7, 1, 0, 0), (257, 129, 8, 0, 1, 1), (300, 100, 12, 0, 0, 0),
    (1411, 1000, 15, 0, 0, 3), (700, 16, 16, 0, 3, 0), (4097, 300, 16, 4, 0, 0), (1000, 255, 23, 0, 0, 0), (5001, 512, 24, 0, 0, 0),
    (4000, 785, 30, 0, 0, 0), (20000, 20, 31, 3, 0, 0), (10007, 128, 32, 0, 0, 0), (70001, 16, 32, 0, 0, 0), (129, 77, 40, 0, 0, 0),
    (3001, 300, 48, 0, 0, 0), (140000, 3, 48, 0, 0, 0), (2000, 100, 56, 0, 0, 0), (9001, 36, 63, 0, 2, 0), (140001, 10, 64, 0, 0, 0),
    (67584, 12, 61, 0, 0, 0), (300001, 20, 15, 0, 0, 0), (60000, 250, 30, 2, 0, 0), (14000, 1000, 15, 0, 0, 0), (33, 514, 64, 0, 0, 0),
    (300000, 10, 50, 0, 0, 0),
]


# those that other kernels take faster
SCANS_LEFT = [(67585, 12, 61, 0, 0, 0), (600000, 2, 30, 0, 0, 0), (600000, 10, 40, 0, 0, 0), (300001, 10, 50, 0, 0, 0)]


@pytest.mark.parametrize("case", SCANS + SCANS_LEFT, ids=lambda c: "N%d_M%d_C%d_p%d_c%d_t%d" % c)
def test_scan_by_blocks(mad, case):
    import torch
    N, M, C, pad, before, at = case
    print("case", case, flush=True)
    rng = np.random.default_rng(N + M + C)
    codes_h = rng.integers(0, 256, size=(N, (C + 1) // 2)).astype(np.uint8)
    if C % 2:
        codes_h[:, -1] &= 15
    luts_h = rng.integers(0, 256, size=(C, 16, M), dtype=np.uint8)
    luts_h[:, :, 0] = 255                           # the largest sums
    raw_codes, raw_luts = (torch.zeros(n, dtype=torch.uint8, device="cuda") for n in (codes_h.size + before, luts_h.size + at))
    raw_codes[before:] = dev(codes_h).reshape(-1)
    raw_luts[at:] = dev(luts_h).reshape(-1)
    codes, luts = raw_codes[before:].reshape(codes_h.shape), raw_luts[at:].reshape(C, 16, M)
    scale, offset = (dev(rng.standard_normal(M).astype(np.float32)) for _ in range(2))

    def run(want_out=True):
        acc = torch.zeros((N, M), dtype=torch.int16, device="cuda") if N < 5000 else None
        full = torch.full((N, M + pad), -3.0, device="cuda")
        mad.maddness_scan(C, codes, luts, scale, offset, out=full[:, :M] if want_out else None, acc=acc, want_out=want_out)
        kernel = mad.maddness_last_kernel()
        torch.cuda.synchronize()
        return full, acc, kernel

    got, got_acc, kernel = run()
    assert kernel.startswith("fused_blocks_kernel, scan") == (case not in SCANS_LEFT), kernel
    only = run(False)[1] if got_acc is not None else None
    try:
        mad.maddness_set_option(mad.MADDNESS_OPT_KERNELS, mad.MADDNESS_KERNELS_GENERAL)
        want, want_acc, kernel = run()
    finally:
        mad.maddness_set_option(mad.MADDNESS_OPT_KERNELS, 0)
    assert kernel.startswith("scan_kernel"), kernel
    assert torch.equal(got, want)
    if got_acc is not None:
        assert torch.equal(got_acc, want_acc) and torch.equal(only, want_acc)
    if N <= 300:
        out, acc, _ = oracle.scan(codes_h, C, luts_h, scale.cpu().numpy(), offset.cpu().numpy())
        assert (got[:, :M].cpu().numpy() == out).all() and (got_acc.cpu().numpy().view(np.uint16) == acc).all()


# (N, D, C, dtype, by columns, elements between rows or columns, elements before the first): every kernel size with and without codebooks
# that do not exist, one chunk to a workgroup and several, rows on any element
CODES = [
    (1, 27, 5, "f16", False, 0, 0), (1, 64, 8, "f32", False, 0, 1), (7, 512, 47, "u8", False, 3, 0), (15, 130, 63, "bf16", False, 0, 1),
    (16, 27, 5, "f16", False, 0, 0), (700, 27, 3, "u8", False, 0, 1), (4099, 130, 8, "u8", False, 3, 1), (100003, 97, 15, "f16", False, 0, 0),
    (30001, 250, 24, "bf16", False, 1, 0), (20000, 120, 30, "f32", False, 0, 0), (9001, 512, 47, "u8", False, 0, 3), (50001, 256, 63, "bf16", False, 0, 0),
    (1025, 33, 8, "f16", True, 0, 0), (1153, 64, 7, "u8", True, 1, 1), (4097, 64, 15, "bf16", True, 0, 1), (200001, 60, 12, "u8", True, 3, 0),
    (30001, 97, 24, "f32", True, 0, 0), (120001, 120, 30, "f16", True, 1, 0), (10001, 190, 48, "f32", True, 0, 1), (70001, 252, 63, "u8", True, 0, 0),
    (70, 40, 8, "f32", False, 0, 0), (13108, 60, 15, "f32", False, 0, 0), (2048, 90, 20, "u8", False, 0, 0), (4506, 90, 20, "u8", False, 0, 0),
    (100001, 27, 3, "f32", False, 0, 1), (8192, 60, 15, "f32", True, 0, 0), (9216, 100, 25, "f32", True, 0, 0), (2048, 64, 8, "f32", False, 0, 0), (4608, 100, 23, "u8", True, 0, 0),
    (16384, 64, 8, "f32", False, 0, 0),
]
# as many codes and fewer, for which the general kernel is the faster one
FEW_CODES = [
    (16, 27, 5, "f32", False, 0, 0), (13107, 60, 15, "f32", False, 0, 0), (2049, 90, 20, "u8", False, 0, 0), (4505, 90, 20, "u8", False, 0, 0),
    (8191, 60, 15, "f32", True, 0, 0), (9215, 100, 25, "f32", True, 0, 0), (2049, 64, 8, "f32", False, 0, 0), (4607, 100, 23, "u8", True, 0, 0), (262145, 40, 12, "f32", True, 0, 0),
    (16383, 64, 8, "f32", False, 0, 0),
]


@pytest.mark.parametrize("case", CODES + FEW_CODES, ids=lambda c: "N%d_D%d_C%d_%s_cols%d_p%d_o%d" % c)
def test_codes_by_blocks(mad, case):
    import torch
    N, D, C, dtype, cols, pad, before = case
    print("case", case, flush=True)
    A, sd, th, _, _, _ = problem(N + D, min(N, 2048), D, 4, C)
    kind = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "u8": torch.uint8}[dtype]
    many, inner = (D, N) if cols else (N, D)
    raw = torch.full((before + many * (inner + pad),), 1, dtype=kind, device="cuda")
    A_d = raw[before:].view(many, inner + pad)[:, :inner]
    values = (dev(A) * (60 if dtype == "u8" else 1)).clamp(max=255).to(kind)[torch.arange(N, device="cuda") % len(A)]
    A_d.copy_(values.t() if cols else values)
    params = mad.Params(dev(sd), dev(th))
    got = mad.maddness_encode_typed(params, A_d, col_major=cols)
    kernel = mad.maddness_last_kernel()
    torch.cuda.synchronize()
    assert kernel.startswith("fused_blocks_kernel, codes of " + ("columns" if cols else "rows")) == (case not in FEW_CODES), kernel
    want = oracle.pack(oracle.encode(values.float().cpu().numpy(), sd, th)) if N <= 5000 else None
    if want is None:
        try:
            mad.maddness_set_option(mad.MADDNESS_OPT_KERNELS, mad.MADDNESS_KERNELS_GENERAL)
            want = mad.maddness_encode_typed(params, A_d, col_major=cols).cpu().numpy()
            assert mad.maddness_last_kernel().startswith("encode_kernel"), mad.maddness_last_kernel()
        finally:
            mad.maddness_set_option(mad.MADDNESS_OPT_KERNELS, 0)
    assert (got.cpu().numpy() == want).all()

"""GPU parity at the edges of three pieces: the tables' way into the registers of the matrix-core scan (any M, any
alignment, few rows), A stored by columns encoded a row to a lane, and the staged product of the table build; and the
learner's ridge solve at the sizes where its launch changes, and its trees on data with infinities.  Codes,
accumulators, outputs, trees and prototypes equal the oracle's to the bit; table bytes as in compare_luts."""
import numpy as np
import pytest

import oracle
from helpers import compare_luts, oracle_pipeline, random_trees

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mad():
    import torch
    import paper_2106_10860_amd as m
    assert torch.cuda.is_available()
    m.lib()
    return m


def dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def problem(seed, N, D, M, C):
    rng = np.random.default_rng(seed)
    A = np.maximum(rng.standard_normal((N, D)), 0).astype(np.float32)
    sd, th = random_trees(rng, A, C)
    luts = rng.integers(0, 256, size=(C, 16, M)).astype(np.uint8)
    scale = np.exp2(-rng.integers(0, 6, size=M)).astype(np.float32)
    offset = rng.standard_normal(M).astype(np.float32)
    return A, sd, th, luts, scale, offset


# (N, D, M, C, bytes the tables start after a 16-byte boundary): tables of more than 64 KiB take the matrix cores from
# the first row on; one row, whole and broken units of 8 and groups of 16, one to three columns after the last four,
# less than four columns in all, padding codebooks, several passes of columns
FEW = [
    (1, 256, 512, 64, 0), (7, 256, 260, 64, 0), (17, 1024, 1032, 32, 0), (33, 128, 1001, 16, 0), (9, 300, 333, 24, 0),
    (65, 300, 342, 24, 1), (255, 512, 255, 30, 3), (300, 512, 1022, 32, 2), (40, 200, 97, 50, 1), (129, 160, 128, 40, 0),
    (16390, 200, 3, 20, 1), (16390, 200, 1, 33, 0), (16385, 256, 2, 64, 0), (16390, 200, 2, 40, 2), (16387, 130, 1, 16, 3),
    (16384, 300, 3, 48, 1), (16384, 140, 2, 5, 0),
]


@pytest.mark.parametrize("shape", FEW, ids=lambda s: "N%d_D%d_M%d_C%d_at%d" % s)
def test_tables_in_registers(mad, shape, blocks):
    import torch
    N, D, M, C, at = shape
    print("case", shape, flush=True)
    A, sd, th, luts, scale, offset = problem(N + D + M, N, D, M, C)
    want_out, want_acc, want_codes = oracle.encode_scan(A, sd, th, luts, scale, offset)
    params = mad.Params(dev(sd), dev(th))
    raw = torch.zeros(luts.size + at, dtype=torch.uint8, device="cuda")
    raw[at:] = dev(luts).reshape(-1)
    luts_d = raw[at:].reshape(C, 16, M)
    acc = torch.zeros((N, M), dtype=torch.int16, device="cuda")
    codes = torch.zeros((N, (C + 1) // 2), dtype=torch.uint8, device="cuda")
    out = mad.maddness_encode_scan(params, dev(A), luts_d, dev(scale), dev(offset), acc=acc, codes=codes)
    kernel = mad.maddness_last_kernel()
    torch.cuda.synchronize()
    assert kernel.startswith("fused_mfma_kernel, A by rows") or (blocks and kernel.startswith("fused_blocks_kernel, A by rows")), kernel
    assert (codes.cpu().numpy() == want_codes).all()
    assert (acc.cpu().numpy().view(np.uint16) == want_acc).all()
    assert (out.cpu().numpy() == want_out).all()
    out2, _ = mad.maddness_scan(C, codes, luts_d, dev(scale), dev(offset))
    torch.cuda.synchronize()
    assert (out2.cpu().numpy() == want_out).all(), mad.maddness_last_kernel()


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16", "u8"])
@pytest.mark.parametrize("shape", [(1, 40, 512, 64, 0), (63, 40, 516, 64, 1), (16385, 64, 68, 16, 3), (4099, 48, 256, 32, 0),
                                   (4097, 40, 512, 64, 5), (40000, 32, 64, 32, 2)], ids=lambda s: "N%d_D%d_M%d_C%d_p%d" % s)
def test_by_columns_few_rows(mad, shape, dtype, blocks):
    import torch
    N, D, M, C, pad = shape
    print("case", shape, dtype, flush=True)
    A, sd, th, luts, scale, offset = problem(N + D, N, D, M, C)
    kind = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "u8": torch.uint8}[dtype]
    full = torch.zeros((D, N + pad), dtype=kind, device="cuda")
    full[:, :N] = (dev(A.T) * (60 if dtype == "u8" else 1)).clamp(max=255).to(kind)
    A_d = full[:, :N]
    values = A_d.float().cpu().numpy().T.copy()
    want_out, want_acc, want_codes = oracle.encode_scan(values, sd, th, luts, scale, offset)
    params = mad.Params(dev(sd), dev(th))
    acc = torch.zeros((N, M), dtype=torch.int16, device="cuda")
    codes = torch.zeros((N, C // 2), dtype=torch.uint8, device="cuda")
    out = mad.maddness_encode_scan_typed(params, A_d, dev(luts), dev(scale), dev(offset), col_major=True, acc=acc, codes=codes)
    kernel = mad.maddness_last_kernel()
    torch.cuda.synchronize()
    assert kernel.startswith("fused_mfma_kernel, A by columns, few rows") or (
        blocks and kernel.startswith("fused_blocks_kernel, A by columns")), kernel
    assert (codes.cpu().numpy() == want_codes).all()
    assert (acc.cpu().numpy().view(np.uint16) == want_acc).all()
    assert (out.cpu().numpy() == want_out).all()


# (N, D, M, C, elements between rows, elements before the first): C of 16 and what is padded to 16, 32 and 64; rows of whole
# pieces and rows that start on any element; results by lane and through LDS; full staging
@pytest.mark.parametrize("dtype", ["f16", "bf16", "u8"])
@pytest.mark.parametrize("shape", [(32768, 256, 64, 16, 0, 0), (32771, 250, 33, 15, 3, 1), (1411, 360, 512, 30, 0, 0),
                                   (999, 505, 257, 31, 7, 5), (4097, 768, 250, 48, 0, 0), (32769, 97, 40, 7, 0, 3),
                                   (777, 1009, 193, 57, 0, 7), (70, 1993, 130, 63, 2, 0)],
                         ids=lambda s: "N%d_D%d_M%d_C%d_p%d_o%d" % s)
def test_narrow_rows_of_any_shape(mad, shape, dtype, blocks):
    import torch
    N, D, M, C, pad, before = shape
    print("case", shape, dtype, flush=True)
    A, sd, th, luts, scale, offset = problem(N + D, N, D, M, C)
    kind = {"f16": torch.float16, "bf16": torch.bfloat16, "u8": torch.uint8}[dtype]
    full = torch.full((before + N * (D + pad),), 1, dtype=kind, device="cuda")
    A_d = full[before:].view(N, D + pad)[:, :D]
    A_d.copy_((dev(A) * (60 if dtype == "u8" else 1)).clamp(max=255).to(kind))
    values = A_d.float().cpu().numpy().copy()
    want_out, want_acc, want_codes = oracle.encode_scan(values, sd, th, luts, scale, offset)
    params = mad.Params(dev(sd), dev(th))
    acc = torch.zeros((N, M), dtype=torch.int16, device="cuda")
    codes = torch.zeros((N, (C + 1) // 2), dtype=torch.uint8, device="cuda")
    out = mad.maddness_encode_scan_typed(params, A_d, dev(luts), dev(scale), dev(offset), acc=acc, codes=codes)
    kernel = mad.maddness_last_kernel()
    torch.cuda.synchronize()
    assert kernel.startswith("fused_mfma_kernel, A by rows") or (blocks and kernel.startswith("fused_blocks_kernel, A by rows")), kernel
    assert (codes.cpu().numpy() == want_codes).all()
    assert (acc.cpu().numpy().view(np.uint16) == want_acc).all()
    assert (out.cpu().numpy() == want_out).all()


@pytest.mark.parametrize("dtype,D,C,M", [("f32", (1 << 29) + 4, 30, 300), ("f32", (1 << 29) + 4, 32, 260),
                                         ("bf16", (1 << 30) + 16, 32, 260), ("bf16", (1 << 30) + 16, 32, 128),
                                         ("u8", (1 << 31) - 9, 24, 400)])
def test_rows_of_more_than_2_gib(mad, dtype, D, C, M):
    """The bytes of such a row do not fit 32 bits (or end just below): no kernel may take it for a short one."""
    import torch
    print("case", dtype, D, C, M, flush=True)
    rng = np.random.default_rng(C + M)
    used = np.unique(np.concatenate([[0, D - 1], rng.integers(0, D, size=60)]))
    values = rng.integers(0, 200, size=(1, len(used))).astype(np.float32)
    sd, th = random_trees(rng, values, C)
    luts = rng.integers(0, 256, size=(C, 16, M)).astype(np.uint8)
    scale, offset = np.ones(M, np.float32), np.zeros(M, np.float32)
    want_out, _, want_codes = oracle.encode_scan(values, sd, th, luts, scale, offset)
    A = torch.zeros((1, D), dtype={"f32": torch.float32, "bf16": torch.bfloat16, "u8": torch.uint8}[dtype], device="cuda")
    A[0, dev(used)] = dev(values)[0].to(A.dtype)
    codes = torch.zeros((1, (C + 1) // 2), dtype=torch.uint8, device="cuda")
    out = mad.maddness_encode_scan_typed(mad.Params(dev(used[sd].astype(np.int32)), dev(th)), A, dev(luts), dev(scale), dev(offset),
                                         codes=codes)
    torch.cuda.synchronize()
    assert (codes.cpu().numpy() == want_codes).all()
    assert (out.cpu().numpy() == want_out).all()


# (N, D, M, C, dtype, by columns) -> the kernel that measured faster, and that of those beside the one by blocks of rows and columns:
# either side of the rules of the dispatch
B, F, G, K = "fused_blocks", "fused_mfma", "scan_kernel", "cols_kernel"
FASTER = [
    # tables between 64 KiB and what the general kernel holds at once: padding of codebooks and columns decides, and rows
    ((1, 1500, 656, 12, "f32", False), B, G), ((239, 1500, 592, 12, "f32", False), B, G),
    ((5257, 510, 300, 16, "f32", False), B, F), ((120, 2001, 340, 16, "f32", False), B, G),
    ((2000, 300, 250, 30, "f32", False), B, F), ((6, 333, 96, 50, "f32", False), B, G),
    ((125, 1000, 288, 20, "f32", False), B, F), ((430, 1500, 780, 12, "bf16", False), B, G),
    ((378, 333, 224, 30, "bf16", False), B, F), ((1, 256, 172, 40, "u8", False), B, G),
    ((16384, 1500, 592, 12, "f32", False), F, F), ((1787, 512, 112, 40, "f32", False), B, G),
    ((1000, 256, 92, 64, "f32", False), B, F), ((1, 256, 72, 64, "f32", False), B, G),
    # narrow rows, small tables: the split values alone or whole rows
    ((32767, 250, 33, 15, "f16", False), B, G), ((32768, 250, 33, 15, "f16", False), B, F),
    ((53325, 85, 20, 16, "u8", False), B, G), ((40000, 716, 5, 4, "u8", False), B, G),
    ((33000, 1558, 92, 2, "f16", False), G, G), ((40001, 174, 8, 22, "bf16", False), B, G),
    ((35000, 426, 42, 53, "u8", False), B, F), ((36000, 472, 66, 16, "bf16", False), B, F),
    ((35550, 107, 72, 16, "f16", False), B, F), ((34561, 901, 23, 32, "u8", False), B, F),
    # rows of many bytes to a codebook
    ((6978, 601, 5, 4, "f32", False), B, G), ((6979, 601, 5, 4, "f32", False), G, G), ((6979, 600, 5, 4, "f32", False), B, G),
    # up to 8 codebooks, several blocks of columns or turns: blocks of rows and columns or whole rows
    ((76800, 136, 768, 8, "f32", False), B, F), ((76801, 136, 768, 8, "f32", False), F, F), ((76801, 79, 768, 8, "f32", False), B, F),
    ((95232, 176, 132, 8, "f32", False), B, F), ((95233, 176, 132, 8, "f32", False), F, F), ((95233, 176, 164, 8, "f32", False), B, F),
    ((131072, 128, 463, 8, "f32", False), B, F), ((131073, 128, 463, 8, "f32", False), F, F),
    ((209715, 24, 500, 8, "u8", False), B, F), ((209716, 24, 500, 8, "u8", False), F, F),
    # A by columns: small tables by the words of their rows, larger ones up to 8192 rows
    ((80000, 40, 8, 16, "f32", True), B, G), ((97000, 20, 16, 16, "f16", True), B, G),
    ((98304, 20, 16, 16, "f16", True), B, F), ((57000, 24, 28, 32, "u8", True), B, G),
    ((24576, 24, 32, 32, "f32", True), B, F), ((24575, 24, 48, 16, "f32", True), B, G),
    ((24576, 24, 188, 16, "f32", True), B, G), ((24577, 24, 188, 16, "f32", True), B, F),
    ((16385, 24, 192, 16, "u8", True), B, F), ((16384, 24, 192, 16, "u8", True), B, G),
    ((16384, 24, 256, 16, "u8", True), B, F),
    ((8192, 50, 192, 32, "f32", True), B, G), ((8193, 50, 192, 32, "bf16", True), B, F),
    ((300, 50, 584, 16, "f32", True), B, G), ((256, 50, 584, 16, "f32", True), B, F),
    ((4096, 50, 96, 64, "u8", True), B, F),
    # A by columns: blocks of rows and columns or whole rows of results, by the workgroups that these make and their turns
    ((20417, 64, 512, 16, "f32", True), B, F), ((20481, 64, 512, 16, "f32", True), F, F),
    ((81920, 128, 128, 32, "f32", True), B, F), ((81921, 128, 128, 32, "f32", True), F, F),
    ((24576, 128, 256, 32, "f32", True), B, F), ((24577, 128, 256, 32, "f32", True), F, F), ((70001, 128, 300, 32, "f32", True), B, F),
    ((32768, 128, 512, 32, "u8", True), B, F), ((32769, 128, 512, 32, "u8", True), F, F), ((32769, 128, 500, 32, "u8", True), B, F),
    ((16384, 256, 64, 64, "f32", True), B, F), ((16385, 256, 64, 64, "f32", True), F, F), ((16385, 256, 128, 64, "f32", True), F, F),
    ((24576, 256, 256, 64, "f16", True), B, F), ((24577, 256, 256, 64, "f16", True), F, F), ((16385, 64, 200, 64, "f16", True), F, F),
    ((98304, 64, 128, 64, "f16", True), B, F), ((98305, 64, 128, 64, "f16", True), F, F),
    ((131077, 64, 256, 16, "f32", True), K, K), ((131077, 64, 192, 16, "f32", True), B, K), ((131076, 64, 192, 16, "f32", True), K, K),
    ((170000, 128, 64, 32, "f32", True), B, F), ((170004, 128, 64, 32, "f32", True), F, F), ((200000, 128, 64, 32, "u8", True), B, F),
    ((200004, 128, 64, 32, "u8", True), F, F), ((200004, 128, 36, 32, "u8", True), B, F), ((131077, 128, 256, 32, "f32", True), K, K),
    ((131076, 256, 96, 64, "f16", True), B, F), ((131076, 256, 64, 64, "f16", True), F, F),
    # numbers of codebooks that only the general kernel has besides, and where that is the faster one
    ((554, 200, 100, 40, "f16", True), B, G), ((49152, 16, 4, 2, "f16", True), B, G), ((49153, 16, 4, 2, "f16", True), G, G),
    ((49153, 16, 9, 2, "f16", True), B, G), ((147456, 24, 8, 6, "f32", True), B, G), ((147457, 24, 8, 6, "f32", True), G, G),
    ((147457, 24, 8, 6, "u8", True), B, G),
]


@pytest.mark.parametrize("case", FASTER, ids=lambda c: "N%d_D%d_M%d_C%d_%s_%d" % c[0])
def test_dispatch_either_side(mad, case, blocks):
    import torch
    (N, D, M, C, dtype, col_major), family, beside = case
    if not blocks:
        family = beside
    print("case", case, flush=True)
    A, sd, th, luts, scale, offset = problem(N + D, N, D, M, C)
    kind = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "u8": torch.uint8}[dtype]
    A_d = (dev(A.T if col_major else A) * (60 if dtype == "u8" else 1)).clamp(max=255).to(kind)
    values = A_d.float().cpu().numpy()
    want_out, _, want_codes = oracle.encode_scan(values.T.copy() if col_major else values, sd, th, luts, scale, offset)
    codes = torch.zeros((N, (C + 1) // 2), dtype=torch.uint8, device="cuda")
    out = mad.maddness_encode_scan_typed(mad.Params(dev(sd), dev(th)), A_d, dev(luts), dev(scale), dev(offset), col_major=col_major,
                                         codes=codes)
    kernel = mad.maddness_last_kernel()
    torch.cuda.synchronize()
    assert kernel.startswith(family), kernel
    assert (codes.cpu().numpy() == want_codes).all()
    assert (out.cpu().numpy() == want_out).all()


# (D, M, C): one tile and parts of tiles of the inner dimension (64), the columns (32 a workgroup, 64 a workgroup of the
# quantisation) and the codebooks (1, 2 or 4 a workgroup, whichever leaves one for every compute unit; 8 minima at a time)
@pytest.mark.parametrize("shape", [(1, 1, 1), (63, 31, 3), (64, 32, 4), (65, 33, 5), (130, 65, 17), (200, 520, 33), (129, 520, 63),
                                   (70, 1030, 255)], ids=lambda s: "D%d_M%d_C%d" % s)
def test_table_build_at_tile_edges(mad, shape):
    import torch
    D, M, C = shape
    print("case", shape, flush=True)
    rng = np.random.default_rng(D + M + C)
    P = rng.standard_normal((C, 16, D)).astype(np.float32)
    B = rng.standard_normal((D, M + 3)).astype(np.float32)
    A = rng.standard_normal((5, D)).astype(np.float32)
    sd, th = random_trees(rng, A, C)
    ref = oracle_pipeline(A, sd, th, P, B[:, :M].copy())
    params = mad.Params(dev(sd), dev(th), dev(P))
    luts, scale, offset = mad.maddness_build_luts(params, dev(B)[:, :M])
    torch.cuda.synchronize()
    compare_luts(luts.cpu().numpy(), scale.cpu().numpy(), offset.cpu().numpy(), ref, P, B[:, :M])


@pytest.mark.parametrize("C", [1, 15, 16, 17, 33, 255])
def test_pooled_table_build_around_a_batch_of_codebooks(mad, C):
    """Whole values, so that the tables are exact; one entry is not a number."""
    import torch
    rng = np.random.default_rng(C)
    P, B = rng.integers(-9, 10, size=(C, 16, 7)).astype(np.float32), rng.integers(-5, 6, size=(7, 11)).astype(np.float32)
    P[C - 1, 3, 2] = np.nan
    want_luts, want_scale, want_offset, _, _ = oracle.quantize_luts_pooled(oracle.build_luts_f64(P, B))
    sd, th = np.zeros((C, 4), np.int32), np.zeros((C, 16), np.float32)
    luts, scale, offset = mad.maddness_build_luts_pooled(mad.Params(dev(sd), dev(th), dev(P)), dev(B))
    torch.cuda.synchronize()
    assert (scale.cpu().numpy() == want_scale).all() and (offset.cpu().numpy() == want_offset).all()
    assert (luts.cpu().numpy() == want_luts).all()


@pytest.mark.parametrize("kind", ["nan", "inf", "mixed"])
def test_table_build_on_prototypes_that_are_not_numbers(mad, kind):
    """One entry after the other of a table is not a number or infinite: the finite ones keep minimum, range and bytes,
    and only a table whose first entry is not a number has none.  Whole values, so that the tables are exact."""
    import torch
    rng = np.random.default_rng(len(kind))
    C, D, M = 19, 5, 33
    P = rng.integers(-9, 10, size=(C, 16, D)).astype(np.float32)
    B = rng.integers(1, 5, size=(D, M)).astype(np.float32)
    for c in range(16):
        P[c, c, c % D] = {"nan": np.nan, "inf": np.inf, "mixed": np.nan if c % 2 else -np.inf}[kind]
    P[16, 1:] = np.nan
    P[17, [2, 7, 9]] = [[np.nan], [np.inf], [-np.inf]]
    P[18] = np.inf if kind == "inf" else np.nan
    # (a codebook at a time too: a column's scale is that of its widest table)
    for first, last in [(0, C)] + [(c, c + 1) for c in range(C)]:
        Pc = np.ascontiguousarray(P[first:last])
        want_luts, want_scale, want_offset, _, _ = oracle.quantize_luts(oracle.build_luts_f64(Pc, B))
        sd, th = np.zeros((last - first, 4), np.int32), np.zeros((last - first, 16), np.float32)
        luts, scale, offset = mad.maddness_build_luts(mad.Params(dev(sd), dev(th), dev(Pc)), dev(B))
        torch.cuda.synchronize()
        assert (scale.cpu().numpy() == want_scale).all(), (first, last)
        assert np.array_equal(offset.cpu().numpy(), want_offset, equal_nan=True), (first, last)
        assert (luts.cpu().numpy() == want_luts).all(), (first, last)


@pytest.mark.parametrize("C", [1, 4, 36, 37, 73, 110])
def test_ridge_solve_where_its_launch_changes(mad, C):
    """One and four panels of 16, and either side of the sizes at which a helper takes more entries of a row (576,
    1152 rows of the factor) or a workgroup fewer columns (1700)."""
    import torch
    rng = np.random.default_rng(C)
    N, D = 300, C + 2
    A = rng.standard_normal((N, D)).astype(np.float32)
    subspaces = [(c, c + 1) for c in range(C)]
    codes = rng.integers(0, 16, size=(N, C)).astype(np.uint8)
    P = mad.maddness_learn_prototypes(dev(codes), dev(A), subspaces, ridge=True, lam=0.5)
    torch.cuda.synchronize()
    assert (P.cpu().numpy() == oracle.ridge_prototypes(codes, A, 0.5).astype(np.float32)).all()


@pytest.mark.parametrize("where", [(0, 5), (3, 5), (700, 700)], ids=["first", "both_signs", "last"])
def test_trees_on_data_with_infinities(mad, where):
    """An infinite value makes the losses of the splits around it not a number; a comparison with one is false, so such a
    split is the best only where it is its bucket's first."""
    import torch
    rng = np.random.default_rng(sum(where))
    A = rng.standard_normal((701, 12)).astype(np.float32)
    A[where[0], 2] = np.inf
    A[where[1], 9] = -np.inf
    subspaces = [(0, 6), (6, 12)]
    sd, th, codes = mad.maddness_learn_trees(dev(A), subspaces)
    torch.cuda.synchronize()
    want_sd, want_th, want_codes, _ = oracle.learn_trees(A, subspaces)
    assert (sd.cpu().numpy() == want_sd).all()
    assert (th.cpu().numpy().view(np.uint32) == want_th.view(np.uint32)).all()
    assert (codes.cpu().numpy() == want_codes).all()


@pytest.mark.parametrize("kind", ["whole", "halves", "leaps", "signed", "tiny", "equal"])
def test_losses_in_row_order(mad, kind):
    """Which columns a level may split rests on the last bits of their losses here: each codebook's columns hold the same
    values in orders of their own.  The kinds take the ways in which the sums are made: exact; half-way cases of the
    rounding in every tile; sums that leave their binade; sums of both signs; the smallest; sums that stay zero."""
    import torch
    rng = np.random.default_rng(len(kind) + ord(kind[0]))
    N, d = 2999, 8
    half = rng.integers(1, 1 << 23, size=N // 2) * 2 + 1                      # odd, 24 bits: squares of 48 bits
    half = np.concatenate([half, -half, [0]]) * 2.0 ** -20                    # of mean exactly 0
    values = {"whole": rng.integers(0, 256, size=N),
              "halves": half,
              "leaps": half * np.exp2(20 * (rng.random(N) < 0.003)),
              "signed": rng.standard_normal(N),
              "tiny": rng.standard_normal(N) * 2.0 ** -140,
              "equal": np.zeros(N)}[kind].astype(np.float32)
    A = np.stack([rng.permutation(values) for _ in range(2 * d)], axis=1)
    if kind == "equal":
        A[:, 3] = rng.permutation(half)
    subspaces = [(0, d), (d, 2 * d)]
    sd, th, codes = mad.maddness_learn_trees(dev(A), subspaces)
    torch.cuda.synchronize()
    want_sd, want_th, want_codes, _ = oracle.learn_trees(A, subspaces)
    assert (sd.cpu().numpy() == want_sd).all()
    assert (th.cpu().numpy().view(np.uint32) == want_th.view(np.uint32)).all()
    assert (codes.cpu().numpy() == want_codes).all()


@pytest.mark.parametrize("width", [5, 20])
@pytest.mark.parametrize("N", [1, 2, 3, 9, 33, 255, 256, 257, 300, 511, 513, 2048, 2049])
def test_trees_of_few_rows(mad, N, width):
    """Buckets of no row, one row and either side of the 256 rows up to which a bucket's sums have a kernel of their own,
    where that kernel is taken and where it is not; skewed, so that a level has both."""
    import torch
    rng = np.random.default_rng(N + width)
    A = np.exp(rng.standard_normal((N, 3 * width))).astype(np.float32)
    A[:, 1] = np.round(A[:, 1])
    A[: N // 2, width] = 1.0
    subspaces = [(0, width), (width, 2 * width), (2 * width, 3 * width)]
    sd, th, codes = mad.maddness_learn_trees(dev(A), subspaces)
    torch.cuda.synchronize()
    want_sd, want_th, want_codes, _ = oracle.learn_trees(A, subspaces)
    assert (sd.cpu().numpy() == want_sd).all()
    assert (th.cpu().numpy().view(np.uint32) == want_th.view(np.uint32)).all()
    assert (codes.cpu().numpy() == want_codes).all()


def test_trees_in_batches(mad):
    """More codebooks than the workspace takes at a time, one of them narrow: the same trees and codes as each alone."""
    import torch
    N, D = 1 << 20, 132
    g = torch.Generator(device="cuda").manual_seed(7)
    A = torch.randn((N, D), device="cuda", generator=g)
    subspaces = [(0, 128), (4, 132), (2, 130), (1, 6), (3, 129), (0, 120), (5, 132)]
    sd, th, codes = mad.maddness_learn_trees(A, subspaces)
    torch.cuda.synchronize()
    for c, subspace in enumerate(subspaces):
        print("codebook", c, flush=True)
        sd1, th1, codes1 = mad.maddness_learn_trees(A, [subspace])
        torch.cuda.synchronize()
        assert torch.equal(sd[c], sd1[0]) and torch.equal(th[c], th1[0]), c
        assert torch.equal(codes[:, c], codes1[:, 0]), c


@pytest.fixture
def options(mad):
    """set_option(option, value) for one test; every switch is back at 0 afterwards."""
    yield mad.maddness_set_option
    for opt in range(4):
        mad.maddness_set_option(opt, 0)


# (N, D, M, C): four rows to a lane from 131073 rows on - whole blocks and a last one in which wavefronts have no rows, and
# rows beyond the last four, which the general kernel takes; a row to a lane below
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16", "u8"])
@pytest.mark.parametrize("shape", [(131076, 20, 128, 32), (133124, 24, 130, 64), (131079, 17, 72, 32), (30001, 20, 128, 32),
                                   (30001, 24, 130, 64), (30001, 24, 132, 16)], ids=lambda s: "N%d_D%d_M%d_C%d" % s)
def test_by_columns_many_blocks(mad, shape, dtype, options):
    """Three workgroups and the fewest rows per block: every workgroup takes many blocks in turn (the area of the codes and
    the one the tables pass through used again, the barrier after the scan)."""
    import torch
    N, D, M, C = shape
    print("case", shape, dtype, flush=True)
    options(mad.MADDNESS_OPT_MAX_WORKGROUPS, 3)
    options(mad.MADDNESS_OPT_PHASED_ROWS, 256)
    A, sd, th, luts, scale, offset = problem(N + D, N, D, M, C)
    kind = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "u8": torch.uint8}[dtype]
    full = torch.zeros((D, (N + 3) // 4 * 4), dtype=kind, device="cuda")
    full[:, :N] = (dev(A.T) * (60 if dtype == "u8" else 1)).clamp(max=255).to(kind)
    A_d = full[:, :N]
    values = A_d.float().cpu().numpy().T.copy()
    want_out, want_acc, want_codes = oracle.encode_scan(values, sd, th, luts, scale, offset)
    acc = torch.zeros((N, M), dtype=torch.int16, device="cuda")
    codes = torch.zeros((N, C // 2), dtype=torch.uint8, device="cuda")
    out = mad.maddness_encode_scan_typed(mad.Params(dev(sd), dev(th)), A_d, dev(luts), dev(scale), dev(offset), col_major=True,
                                         acc=acc, codes=codes)
    kernel = mad.maddness_last_kernel()
    torch.cuda.synchronize()
    assert kernel.startswith("fused_mfma_kernel, A by columns"), kernel
    assert ("few rows" in kernel) == (N < 131073), kernel
    assert (codes.cpu().numpy() == want_codes).all()
    assert (acc.cpu().numpy().view(np.uint16) == want_acc).all()
    assert (out.cpu().numpy() == want_out).all()


@pytest.mark.parametrize("seed", range(4))
def test_selected_kernels_against_general_kernels_at_their_lines(mad, seed, options, blocks):
    """Random shapes with rows on either side of every line of the dispatch, odd widths, columns or rows that start on any
    element: whatever kernel the library selects gives the bits of its general kernels."""
    import torch
    rng = np.random.default_rng(100 + seed)
    rows = [1, 7, 8, 9, 63, 256, 257, 500, 4095, 4096, 8192, 8193, 16383, 16384, 24576, 32767, 32768, 57344, 65536, 98304, 131072, 131073,
            131076]
    kinds = [torch.float32, torch.float32, torch.float16, torch.bfloat16, torch.uint8]
    for case in range(90):
        N, C = int(rng.choice(rows)), int(rng.choice([16, 32, 64, 64, 8, 24, 40, 1, 15, 30, 50]))
        D = int(rng.choice([33, 64, 97, 250, 256, 333, 1021]))
        M = int(rng.choice([1, 2, 3, 8, 16, 20, 33, 64, 68, 128, 132, 255, 256, 260, 300, 333, 512, 584, 1022]))
        if N > 60000: D = int(rng.choice([33, 64, 97]))
        if N > 30000: M = min(M, 300)
        col, kind = bool(rng.random() < 0.45), kinds[int(rng.integers(len(kinds)))]
        pad, before = int(rng.choice([0, 0, 1, 2, 3, 5, 7, 8])), int(rng.choice([0, 0, 0, 1, 2, 3, 5]))
        want_acc, want_codes = bool(rng.random() < 0.4), bool(rng.random() < 0.5)
        print("case", seed, case, N, D, M, C, kind, col, pad, before, want_acc, want_codes, flush=True)
        g = torch.Generator(device="cuda").manual_seed(int(rng.integers(1 << 30)))
        r, c = (D, N) if col else (N, D)
        flat = torch.zeros(before + r * (c + pad), dtype=kind, device="cuda")
        A = flat[before:].view(r, c + pad)[:, :c]
        A.copy_((torch.randn((r, c), device="cuda", generator=g) * (40 if kind == torch.uint8 else 1) +
                 (128 if kind == torch.uint8 else 0)).clamp(-200, 255).to(kind))
        sd = torch.randint(0, D, (C, 4), dtype=torch.int32, device="cuda", generator=g)
        th = torch.randn((C, 16), device="cuda", generator=g) * (30 if kind == torch.uint8 else 0.7) + (128 if kind == torch.uint8 else 0)
        luts = torch.randint(0, 256, (C, 16, M), dtype=torch.uint8, device="cuda", generator=g)
        scale, offset = 2.0 ** torch.randint(-5, 3, (M,), device="cuda", generator=g).float(), torch.randn(M, device="cuda", generator=g)
        params = mad.Params(sd, th)

        def run():
            acc = torch.zeros((N, M), dtype=torch.int16, device="cuda") if want_acc else None
            codes = torch.zeros((N, (C + 1) // 2), dtype=torch.uint8, device="cuda") if want_codes else None
            out = mad.maddness_encode_scan_typed(params, A, luts, scale, offset, col_major=col, acc=acc, codes=codes)
            kernel = mad.maddness_last_kernel()
            enc = mad.maddness_encode_typed(params, A, col_major=col)
            scan, _ = mad.maddness_scan(C, enc, luts, scale, offset)
            torch.cuda.synchronize()
            return [out.view(torch.int32), acc, codes, enc, scan.view(torch.int32)], kernel

        options(mad.MADDNESS_OPT_KERNELS, mad.MADDNESS_KERNELS_AUTO)
        got, kernel = run()
        options(mad.MADDNESS_OPT_KERNELS, mad.MADDNESS_KERNELS_GENERAL)
        want, _ = run()
        for name, x, y in zip(("fused out", "acc", "fused codes", "codes", "scan out"), got, want):
            assert x is None or torch.equal(x, y), f"{name} differs ({kernel})"
        assert torch.equal(got[0], got[4])

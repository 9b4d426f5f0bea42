"""GPU parity of the learning step (maddness_learn_trees / maddness_learn_prototypes, called
through the C ABI) against the oracle's plain statement of Algorithms 2-4 and of the ridge
step on the same seeded training matrices.  Split columns and training codes are integers
and must be equal; thresholds are fp32 midpoints of two data values and must be equal; the
prototypes come out of an fp64 Cholesky solve whose operations run in the oracle's order
and are compared to 1e-6 relative (of the largest entry), with the number of entries that
differ at all reported."""
import ctypes

import numpy as np
import pytest

import oracle
import workloads as wl

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


def check_against_oracle(mad, A, subspaces, label, lda_pad=0, lam=1.0):
    import torch
    N, D = A.shape
    full = torch.zeros((N, D + lda_pad), dtype=torch.float32, device="cuda")
    full[:, :D] = dev(A)
    A_d = full[:, :D]
    sd, th, codes = mad.maddness_learn_trees(A_d, subspaces)
    torch.cuda.synchronize()
    want_sd, want_th, want_codes, _ = oracle.learn_trees(A, subspaces)
    assert (sd.cpu().numpy() == want_sd).all(), f"{label}: split columns differ\n{sd.cpu().numpy()}\n{want_sd}"
    assert (th.cpu().numpy() == want_th).all(), f"{label}: thresholds differ"
    assert (codes.cpu().numpy() == want_codes).all(), f"{label}: training codes differ"
    for ridge in (True, False):
        P = mad.maddness_learn_prototypes(codes, A_d, subspaces, ridge=ridge, lam=lam)
        torch.cuda.synchronize()
        want = oracle.ridge_prototypes(want_codes, A, lam) if ridge else oracle.bucket_means(want_codes, A, subspaces)
        got = P.cpu().numpy()
        tol = 1e-6 * max(np.abs(want).max(), 1e-30)
        assert np.abs(got - want).max() <= tol, f"{label}: prototypes (ridge={ridge}) differ by {np.abs(got - want).max()}"
        print(f"{label}: ridge={ridge}: {(got != want.astype(np.float32)).sum()} of {got.size} prototype entries "
              "differ from the oracle's fp32 rounding", flush=True)
    return sd, th, codes


def even(D, C):
    w = D // C
    return [(c * w, (c + 1) * w) for c in range(C)]


SMALL = [
    # (seed, N, D, subspaces, kind, lda_pad)
    (1, 300, 24, [(0, 8), (8, 16), (16, 24)], "relu", 0),
    (2, 1000, 27, [(0, 7), (7, 14), (14, 21), (21, 27)], "integers", 5),      # the image workload's subspaces
    (3, 65, 10, [(0, 2), (2, 3), (3, 5), (5, 10)], "integers", 0),            # widths 2, 1, 2, 5; one tile + 1 row
    (4, 4097, 64, even(64, 8), "relu", 0),                                    # a row more than a power of two
    (5, 8192, 32, even(32, 2), "normal", 3),                                  # exactly one sort chunk
    (6, 20000, 128, even(128, 2), "relu", 0),                                 # subspaces 64 columns wide, keys in 4 chunks
    (7, 700, 128, [(0, 128)], "normal", 0),                                   # the widest subspace the learner takes
    (8, 50, 5, [(0, 2), (2, 3), (3, 5)], "few_values", 0),                    # buckets that cannot be split, empty buckets
    (9, 1, 4, [(0, 4)], "normal", 0),                                         # one training row
    (10, 9, 2, [(0, 2)], "constant", 0),
    (11, 3000, 48, [(0, 48), (0, 16), (8, 40)], "relu", 0),                   # overlapping subspaces are allowed
    (12, 2000, 100, [(0, 100)], "normal", 0),                                 # the widest kind whose tiles stay in bucket order
    (13, 1500, 66, [(0, 33), (33, 66)], "relu", 1),                           # an odd width, tiles of 128 positions
    (14, 5000, 40, [(0, 3), (3, 40)], "integers", 0),                         # many equal values: ties among the candidate splits
    (15, 600, 224, even(224, 224), "normal", 0),                              # 224 codebooks: a factor of 3584 rows, the substitution kernel for large factors
]


def training_matrix(seed, N, D, kind):
    rng = np.random.default_rng(seed)
    if kind == "relu":
        _, A, _ = wl.random_problem(seed, N, D, 4, latent=min(8, D), N_train=4)
        return A
    if kind == "integers":
        return rng.integers(0, 256, size=(N, D)).astype(np.float32)
    if kind == "few_values":
        return rng.integers(0, 4, size=(N, D)).astype(np.float32)
    if kind == "constant":
        return np.full((N, D), 3.0, dtype=np.float32)
    return rng.standard_normal((N, D)).astype(np.float32)


@pytest.mark.parametrize("case", SMALL, ids=lambda c: "seed%d_N%d_D%d_%s" % (c[0], c[1], c[2], c[4]))
def test_learner_small_cases(mad, case):
    seed, N, D, subspaces, kind, pad = case
    print("case learn", case, flush=True)
    A = training_matrix(seed, N, D, kind)
    sd, th, codes = check_against_oracle(mad, A, subspaces, str(case), lda_pad=pad, lam=1.0 if seed % 2 else 0.5)
    # the learned parameters drive the library's encoder to the same leaves
    import torch
    params = mad.Params(sd, th)
    packed = mad.maddness_encode(params, dev(A))
    torch.cuda.synchronize()
    assert (packed.cpu().numpy() == oracle.pack(codes.cpu().numpy())).all()


def test_learner_random_small_problems(mad):
    """Forty seeded problems of mixed shapes: 1 to 33 codebooks (both launch shapes of the split search), subspaces 1
    to 69 columns wide, 1 to 5000 rows around the tile sizes, continuous data and data with many ties; trees, training
    codes, ridge prototypes and bucket means all equal to the oracle's, to the bit."""
    import torch
    rng = np.random.default_rng(2106)
    for case in range(40):
        C = int(rng.choice([1, 2, 3, 5, 8, 15, 16, 17, 20, 33]))
        widths = rng.integers(1, 12, size=C)
        if rng.random() < 0.2:
            widths[rng.integers(0, C)] = int(rng.integers(30, 70))
        D = int(widths.sum())
        starts = np.concatenate([[0], np.cumsum(widths)[:-1]])
        subspaces = [(int(s), int(s + w)) for s, w in zip(starts, widths)]
        N = int(rng.choice([1, 2, 7, 63, 64, 65, 255, 256, 257, 511, 1000, 2049, 5000]))
        kind = str(rng.choice(["normal", "integers", "few_values"]))
        A = training_matrix(int(rng.integers(1 << 30)), N, D, kind)
        pad = int(rng.integers(0, 4))
        lam = float(rng.choice([1.0, 0.5, 3.0]))
        label = f"case {case}: N={N} D={D} C={C} {kind} pad={pad} lambda={lam}"
        print(label, flush=True)
        full = torch.zeros((N, D + pad), dtype=torch.float32, device="cuda")
        full[:, :D] = dev(A)
        A_d = full[:, :D]
        sd, th, codes = mad.maddness_learn_trees(A_d, subspaces)
        torch.cuda.synchronize()
        want_sd, want_th, want_codes, _ = oracle.learn_trees(A, subspaces)
        assert (sd.cpu().numpy() == want_sd).all(), label
        assert (th.cpu().numpy() == want_th).all(), label
        assert (codes.cpu().numpy() == want_codes).all(), label
        P = mad.maddness_learn_prototypes(codes, A_d, subspaces, ridge=True, lam=lam)
        Pm = mad.maddness_learn_prototypes(codes, A_d, subspaces, ridge=False)
        torch.cuda.synchronize()
        assert (P.cpu().numpy() == oracle.ridge_prototypes(want_codes, A, lam).astype(np.float32)).all(), label
        assert (Pm.cpu().numpy() == oracle.bucket_means(want_codes, A, subspaces).astype(np.float32)).all(), label


@pytest.mark.parametrize("cfg", [1, 2, 3, 4, 5, 6])
def test_learner_on_the_workloads(mad, cfg):
    """The training sets of all six workloads at their full sizes."""
    w = wl.get_workload(cfg)
    print("workload", w.name, flush=True)
    A = wl.make_A_train(w)
    check_against_oracle(mad, A, list(w.subspaces), w.name)


def test_learn_on_device_feeds_the_inference_calls(mad):
    """Learn on the device, build the tables, run the fused call: equal to the oracle fed with the
    oracle-learned parameters."""
    import torch
    w = wl.get_workload(2)
    At, A, B = wl.make_A_train(w), wl.make_A(w), wl.make_B(w)
    params = mad.learn_on_device(dev(At), list(w.subspaces))
    luts, scale, offset = mad.maddness_build_luts(params, dev(B))
    out = mad.maddness_encode_scan(params, dev(A), luts, scale, offset)
    torch.cuda.synchronize()
    sd, th, codes, _ = oracle.learn_trees(At, list(w.subspaces))
    P = oracle.ridge_prototypes(codes, At, 1.0).astype(np.float32)
    assert (params.prototypes.cpu().numpy() == P).all() or np.abs(params.prototypes.cpu().numpy() - P).max() <= 1e-6 * np.abs(P).max()
    want, _, _ = oracle.encode_scan(A, sd, th, luts.cpu().numpy(), scale.cpu().numpy(), offset.cpu().numpy())
    assert (out.cpu().numpy() == want).all()


def test_learner_rejects_bad_arguments(mad):
    import torch
    L = mad.lib()
    A = torch.zeros((100, 300), dtype=torch.float32, device="cuda")
    out_i = torch.zeros((1, 4), dtype=torch.int32, device="cuda")
    out_f = torch.zeros((1, 16), dtype=torch.float32, device="cuda")
    ws = torch.zeros(1 << 22, dtype=torch.uint8, device="cuda")

    def trees(bounds, N=100, D=300, C=1, lda=300):
        b = (ctypes.c_int32 * len(bounds))(*bounds)
        return L.maddness_learn_trees(A.data_ptr(), N, lda, D, C, b, out_i.data_ptr(), out_f.data_ptr(), None,
                                      ws.data_ptr(), ws.numel(), None)
    assert trees([0, 16]) == mad.MADDNESS_OK
    assert trees([0, 129]) == mad.MADDNESS_E_UNSUPPORTED and "128" in L.maddness_last_error().decode()
    assert trees([5, 5]) == mad.MADDNESS_E_INVAL
    assert trees([-1, 4]) == mad.MADDNESS_E_INVAL
    assert trees([290, 301]) == mad.MADDNESS_E_INVAL
    assert trees([0, 16], N=0) == mad.MADDNESS_E_INVAL
    assert trees([0, 16], lda=299) == mad.MADDNESS_E_INVAL
    b = (ctypes.c_int32 * 2)(0, 16)
    assert L.maddness_learn_trees(A.data_ptr(), 100, 300, 300, 1, b, out_i.data_ptr(), out_f.data_ptr(), None, ws.data_ptr(), 64,
                                  None) == mad.MADDNESS_E_UNSUPPORTED
    codes = torch.zeros((100, 1), dtype=torch.uint8, device="cuda")
    P = torch.zeros((1, 16, 300), dtype=torch.float32, device="cuda")
    assert L.maddness_learn_prototypes(codes.data_ptr(), A.data_ptr(), 100, 300, 300, 1, b, 1, 0.0, P.data_ptr(), ws.data_ptr(),
                                       ws.numel(), None) == mad.MADDNESS_E_INVAL
    assert L.maddness_learn_prototypes(None, A.data_ptr(), 100, 300, 300, 1, b, 1, 1.0, P.data_ptr(), ws.data_ptr(),
                                       ws.numel(), None) == mad.MADDNESS_E_INVAL
    torch.cuda.synchronize()


def estimate_matrix(N, widths, scale, kinds):
    rng = np.random.default_rng(N)

    def near_copies(n, which):
        """A second half like the first, of which those columns have two rows exchanged."""
        x = np.tile(np.maximum(rng.standard_normal((n[0], (n[1] + 1) // 2)), 0), 2)[:, :n[1]]
        for j in which:
            a, b = np.argsort(x[:, j])[[-1, n[0] // 4]]
            x[[a, b], j] = x[[b, a], j]
        return x
    relu = lambda n: np.maximum(rng.standard_normal(n), 0)
    draw = {"i": lambda n: rng.integers(0, 256, n), "s": lambda n: rng.integers(-300, 300, n), "w": lambda n: rng.integers(0, 1 << 17, n),
            "W": lambda n: rng.integers(0, 1 << 20, n), "r": relu, "c": lambda n: np.where(rng.random(n) < 0.999, 7, 8),
            "d": lambda n: np.tile(relu((n[0], (n[1] + 1) // 2)), 2)[:, :n[1]], "b": lambda n: rng.integers(0, 2, n),
            "n": lambda n: near_copies(n, range(n[1] // 2)), "D": lambda n: near_copies(n, [0]),
            "z": np.zeros, "1": lambda n: np.full(n, 0.1), "o": lambda n: 1000 + 1e-3 * rng.standard_normal(n),
            "h": lambda n: 1e30 * rng.standard_normal(n), "t": lambda n: 1e-41 * rng.standard_normal(n),
            "x": lambda n: np.where(rng.random(n) < 3 / n[0], np.inf, rng.standard_normal(n))}
    return np.concatenate([draw[k]((N, w)) * scale for w, k in zip(widths, kinds)], 1).astype(np.float32)


# settled: per codebook, whether estimates settle all levels' columns and splits (e) or exact sums some (x); both numbers of levels
# where they are known
@pytest.mark.parametrize("N, widths, scale, kinds, settled", [
    (4097, (3, 4, 5), 0.25, "iri", "eee"),       # quarters; a codebook beside them whose sums depend on their order
    (9000, (40, 17), 1.0, "sw", "ee"),           # both signs; values of 17 bits: 2 x 18 + 14 bits, next to the limit of exact sums
    (8500, (5, 2), 1.0, "Ww", "ee"),             # 20 bits: past it
    (270000, (2, 3), 1.0, "ci", "?e"),           # more groups of 256 rows than a workgroup scans at once; equal rows
    (3072, (6, 5), 1.0, "dr", "ee"),             # columns that are copies
    (5003, (6, 9, 65), 1.0, "nDd", "xxe"),       # copies but for one row; a copy of a column and one but for one row
    (3071, (8, 5), 1.0, "ri", "xx"),             # few rows for columns as few
    (2047, (9, 5), 1.0, "ri", "xx"),
    (700, (4, 3, 2), 1.0, "bz1", "xxx"),         # buckets that cannot be split, columns of zeros, columns of one value
    (3600, (4, 3, 2), 1.0, "bz1", "?ee"),        # the same with estimates
    (2050, (18, 33), 1.0, "dr", "ee"),           # copies in subspaces of more than 16 columns
    (3200, (5, 6, 7), 1.0, "oht", "xee"),        # little spread far from 0; large values; subnormal ones
    (2048, (4, 9), 1.0, "xr", "xe"),             # infinities: comparisons with what is not a number
])
def test_learner_estimates_and_exact_sums(mad, N, widths, scale, kinds, settled):
    """Data whose choices the estimates settle and data that take the exact sums, codebook by codebook: all equal to the oracle's."""
    import torch
    print("case estimates", N, widths, flush=True)
    A = estimate_matrix(N, widths, scale, kinds)
    ends = np.cumsum(widths)
    subspaces = [(int(e - w), int(e)) for e, w in zip(ends, widths)]
    workspace = torch.zeros(mad.lib().maddness_learn_trees_workspace(N, A.shape[1], len(widths), mad._bounds(subspaces)[0]),
                            dtype=torch.uint8, device="cuda")
    sd, th, codes = mad.maddness_learn_trees(dev(A), subspaces, workspace=workspace)
    by_exact = workspace[:8 * len(widths)].view(torch.int32).cpu().numpy().reshape(-1, 2)
    print("levels by exact sums", by_exact.tolist(), flush=True)
    for kind, levels in zip(settled, by_exact):
        assert kind == "?" or (levels.sum() > 0) == (kind == "x") and (levels <= 4).all(), by_exact
    if N < (3072 if max(widths) <= 8 else 2048):
        assert (by_exact == 4).all()
    P = mad.maddness_learn_prototypes(codes, dev(A), subspaces)
    want_sd, want_th, want_codes, _ = oracle.learn_trees(A, subspaces)
    assert (sd.cpu().numpy() == want_sd).all()
    assert (th.cpu().numpy().view(np.uint32) == want_th.view(np.uint32)).all()
    assert (codes.cpu().numpy() == want_codes).all()
    if not np.isfinite(A).all():
        return
    want = oracle.ridge_prototypes(want_codes, A, 1.0)
    # the same fp64 operations: both round to the same fp32
    assert (P.cpu().numpy() == want.astype(np.float32)).all()


@pytest.mark.parametrize("C, widths", [(1, (70,)), (3, (9, 64, 3))], ids=str)
def test_prototypes_of_shared_rows(mad, C, widths):
    """G^T A~ by several wavefronts to a code, over more rows than are listed at a time: codes that only some of the lists hold
    or none, 64 columns of whole values beside columns whose sums depend on their order."""
    N, D = 70001, 130
    rng = np.random.default_rng(C)
    print("case shared rows", C, flush=True)
    A = rng.integers(-100, 100, (N, D)).astype(np.float32)
    A[:, 64:128] = rng.standard_normal((N, 64))
    codes = rng.integers(0, 16, (N, C)).astype(np.uint8)
    codes[:, 0] = np.sort(codes[:, 0])
    codes[codes == 5] = 6
    P = mad.maddness_learn_prototypes(dev(codes), dev(A), [(0, w) for w in widths])
    want = oracle.ridge_prototypes(codes, A, 1.0)
    assert (P.cpu().numpy() == want.astype(np.float32)).all()


@pytest.mark.parametrize("N", [2, 63, 64, 65, 129, 511, 512, 513])
def test_learner_sorts_few_rows(mad, N):
    """Either side of the rows that are sorted by counting: values that repeat, both zeros, both signs."""
    rng = np.random.default_rng(N)
    print("case few rows", N, flush=True)
    A = np.concatenate([rng.standard_normal((N, 5)), rng.integers(-2, 3, (N, 6)) * 0.5, np.where(rng.random((N, 3)) < 0.5, -0.0, 0.0)], 1).astype(np.float32)
    check_against_oracle(mad, A, [(0, 5), (5, 11), (8, 14), (11, 14)], f"few rows {N}")

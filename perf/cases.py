"""The calls a program makes through this package, over the sizes it makes them at.

A case names one public call, its sizes and the kind of data; everything else follows from a seed.
What the calls stand for:

  * ``encode_scan`` - the approximate product of one batch with a fixed matrix, the call a serving loop makes
    (fp32 rows; binary16 / bfloat16 / uint8 rows or A stored by columns through the typed entry point);
  * ``encode`` and ``scan`` - the two halves, where codes are kept (an index, a cache of activations) and
    scanned later, perhaps against several matrices;
  * ``averaged`` - the product with the paper's aggregation by pairwise averages;
  * ``tables`` - h(B), made again whenever the matrix changes;
  * ``learn`` - trees and ridge prototypes from a training matrix that is already on the device.

Sizes and data are those of this repository's workloads (softmax layers of 512 features, 3x3 windows of an
image, series of length 320, the throughput and stress shapes) and of the odd shapes its tests use.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2106_10860_amd as m

DEVICE = "cuda"
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "u8": torch.uint8}
PIECE = 65536          # rows of A made, or checked, at a time


def _case(name, call, N, D, M, C, data="relu", dtype="f32", columns=False):
    return {"name": name, "call": call, "N": N, "D": D, "M": M, "C": C, "data": data, "dtype": dtype, "columns": columns}


def listed():
    return [
        # a small batch of series against 128 exemplars: one request of a nearest-exemplar service
        _case("series_request", "encode_scan", 1000, 320, 128, 16, data="series"),
        # a test set of 10^4 activations through a 100-way softmax layer
        _case("softmax_100", "encode_scan", 10000, 512, 100, 32),
        # every 3x3 window of a 512 x 512 RGB image against two filters
        _case("image_filters", "encode_scan", 260100, 27, 2, 4, data="image"),
        # the throughput shape: 2^20 rows of 512 features, 256 outputs
        _case("throughput", "encode_scan", 1 << 20, 512, 256, 32),
        # the largest one: 24 GiB of rows and results, tables larger than a compute unit's on-chip memory
        _case("stress", "encode_scan", 1 << 22, 1024, 512, 64),
        # nothing a multiple of anything
        _case("ragged", "encode_scan", 300007, 510, 250, 30),
        # hidden states in bfloat16, a prefill's worth of rows, a wide layer
        _case("hidden_states_bf16", "encode_scan", 65536, 1024, 512, 64, dtype="bf16"),
        # a column store of half-precision features, codes kept for later scans
        _case("encode_columns_f16", "encode", 1 << 20, 512, 0, 32, dtype="f16", columns=True),
        # stored codes against the 1000 columns of a classifier
        _case("scan_classes", "scan", 131072, 0, 1000, 32),
        # the tables of a 1024 x 512 layer
        _case("tables_layer", "tables", 0, 1024, 512, 64),
        # trees and prototypes from 20000 activations of 512 features
        _case("learn_activations", "learn", 20000, 512, 0, 32),
        # trees and prototypes from the windows of one image
        _case("learn_image", "learn", 260100, 27, 0, 4, data="image"),
    ]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["encode_scan"] * 6 + ["typed"] * 3 + ["encode", "scan", "averaged", "tables"] + ["learn"] * 2)
    C = rng.choice([4, 8, 15, 16, 16, 24, 30, 32, 32, 32, 48, 64, 64])
    D = rng.choice([C * _spread(rng, 4, 32), C * rng.choice([8, 16, 16, 32]), C * rng.choice([8, 16])])
    M = rng.choice([_spread(rng, 2, 1024), rng.choice([10, 100, 128, 256, 512, 1000])])
    N = rng.choice([_spread(rng, 500, 1 << 20), _spread(rng, 500, 1 << 20), 1 << rng.randint(10, 20)])
    data, dtype, columns = "relu", "f32", False
    if call == "typed":
        call, dtype, columns = "encode_scan", rng.choice(["f16", "bf16", "bf16", "u8", "f32"]), rng.random() < 0.4
        columns = columns or dtype == "f32"
    elif call == "encode":
        M, dtype, columns = 0, rng.choice(["f32", "f32", "f16", "bf16", "u8"]), rng.random() < 0.3
    elif call == "scan":
        D = 0
    elif call == "averaged":
        C = rng.choice([16, 32, 64])
        D = C * rng.choice([8, 16, 16])
    elif call == "tables":
        N = 0
    elif call == "learn":
        M, N, C = 0, _spread(rng, 1000, 40000), rng.choice([4, 8, 15, 16, 32, 32, 64])
        D = C * rng.randint(4, 20)
        data = rng.choice(["relu", "relu", "series"])
    elif C == 4:
        D, data = 27, "image"
    elif C == 16 and rng.random() < 0.3:
        D, data = 320, "series"
    case = _case("", call, N, D, M, C, data, dtype, columns)
    del case["name"]
    return case


# ---------------------------------------------------------------------------------------------------------
# inputs

def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return g


def _image_rows(g, N):
    """The first N of the 3x3 windows (channels, then rows, then columns) of a smooth RGB image of whole values 0..255."""
    side = math.isqrt(max(N - 1, 0)) + 1 + 2
    img = torch.rand((3, side, side), generator=g, device=DEVICE)
    kernel = [math.exp(-0.5 * (t / 3.0) ** 2) for t in range(-9, 10)]
    for dim in (1, 2):
        pad = torch.cat([img.narrow(dim, 0, 9).flip(dim), img, img.narrow(dim, side - 9, 9).flip(dim)], dim) if side >= 9 else img
        if pad is not img:
            img = sum(w * pad.narrow(dim, t, side) for t, w in enumerate(kernel))
    lo, hi = img.amin((1, 2), keepdim=True), img.amax((1, 2), keepdim=True)
    img = ((img - lo) / (hi - lo) * 255).round()
    return img.unfold(1, 3, 1).unfold(2, 3, 1).permute(1, 2, 0, 3, 4).reshape(-1, 27)[:N].contiguous()


def _series_rows(g, N, D):
    """Series of eight classes of four sinusoids each, shifted in time, with noise; every row of mean 0 and deviation 1."""
    freq, phase = torch.rand((8, 4), generator=g, device=DEVICE) * 5.5 + 0.5, torch.rand((8, 4), generator=g, device=DEVICE) * 6.283
    amp = torch.rand((8, 4), generator=g, device=DEVICE) * 0.7 + 0.3
    cls = torch.randint(0, 8, (N,), generator=g, device=DEVICE)
    t = torch.arange(D, device=DEVICE) / D + (torch.rand((N, 1), generator=g, device=DEVICE) - 0.5) * 0.1
    X = 0.2 * torch.randn((N, D), generator=g, device=DEVICE)
    for h in range(4):
        X += amp[cls, h][:, None] * torch.sin(6.2831853 * freq[cls, h][:, None] * t + phase[cls, h][:, None])
    X -= X.mean(1, keepdim=True)
    return X / X.std(1, keepdim=True)


def _matrix(case, g):
    """A (or the training matrix) as the call takes it: [N][D], or [D][N] where it is stored by columns."""
    N, D, dtype = case["N"], case["D"], DTYPES[case["dtype"]]
    if case["data"] == "image":
        rows = _image_rows(g, N)
        rows = rows.to(dtype)
        return rows.t().contiguous() if case["columns"] else rows
    if case["data"] == "series":
        rows = _series_rows(g, N, D).to(dtype)
        return rows.t().contiguous() if case["columns"] else rows
    # activations after a ReLU, of a low-dimensional origin: max(0, Z W + noise)
    W = torch.randn((64, D), generator=g, device=DEVICE) / 8
    A = torch.empty((D, N) if case["columns"] else (N, D), dtype=dtype, device=DEVICE)
    for lo in range(0, N, PIECE):
        n = min(PIECE, N - lo)
        rows = torch.randn((n, 64), generator=g, device=DEVICE) @ W
        rows += 0.1 * torch.randn((n, D), generator=g, device=DEVICE)
        rows.clamp_(min=0)
        if dtype == torch.uint8:
            rows = (rows * 64).round_().clamp_(max=255)
        if case["columns"]:
            A[:, lo:lo + n] = rows.t().to(dtype)
        else:
            A[lo:lo + n] = rows.to(dtype)
    return A


def _subspaces(D, C):
    return [(c * D // C, (c + 1) * D // C) for c in range(C)]


def _trees(case, A, seed):
    """Trees that split a sample of the rows evenly: at every level a column of the codebook's subspace, at every
    node the mean of its rows there (half-way between two values of the data, so that few rows tie)."""
    rng = np.random.default_rng(seed)
    X = (A[:, :2048].t() if case["columns"] else A[:2048]).float().cpu().numpy()
    C = case["C"]
    dims, thresholds = np.zeros((C, 4), np.int32), np.zeros((C, 16), np.float32)
    for c, (lo, hi) in enumerate(_subspaces(case["D"], C)):
        dims[c] = lo + (rng.permutation(hi - lo)[np.arange(4) % (hi - lo)])
        node = np.zeros(len(X), np.int64)
        for t in range(4):
            x, first = X[:, dims[c, t]], (1 << t) - 1
            count = np.maximum(np.bincount(node, minlength=1 << t), 1)
            v = (np.bincount(node, x, minlength=1 << t) / count).astype(np.float32)
            thresholds[c, first:first + (1 << t)] = v
            node = 2 * node + (x >= v[node])
    return torch.from_numpy(dims).to(DEVICE), torch.from_numpy(thresholds).to(DEVICE)


def _tables(C, M, g):
    """Tables as the quantisation leaves them: every codebook's least entry 0 in each column, a power-of-two scale."""
    T = torch.randn((C, 16, M), generator=g, device=DEVICE)
    delta = T.amin(1, keepdim=True)
    widest = (T - delta).amax((0, 1))
    scale = torch.exp2(torch.ceil(torch.log2(widest / 255)))
    return ((T - delta) / scale).round().clamp(0, 255).to(torch.uint8), scale, delta.sum((0, 1)).contiguous()


def prepare(case, seed):
    g = _generator(seed)
    call, N, D, M, C = (case[k] for k in ("call", "N", "D", "M", "C"))
    state = {"case": case}
    if call == "learn":
        state.update(A=_matrix(case, g), subspaces=_subspaces(D, C))
        return state
    if call == "tables":
        # dense prototypes, as the ridge step leaves them: largest on the codebook's own columns
        P = 0.05 * torch.randn((C, 16, D), generator=g, device=DEVICE)
        for c, (lo, hi) in enumerate(_subspaces(D, C)):
            P[c, :, lo:hi] += torch.randn((16, hi - lo), generator=g, device=DEVICE).clamp(min=0)
        state["B"] = torch.randn((D, M), generator=g, device=DEVICE) / math.sqrt(D)
        state["params"] = m.Params(torch.zeros((C, 4), dtype=torch.int32, device=DEVICE),
                                   torch.zeros((C, 16), device=DEVICE), P)
        return state
    if call != "encode":
        state["luts"], state["scale"], state["offset"] = _tables(C, M, g)
    if call == "scan":
        codes = torch.randint(0, 256, (N, (C + 1) // 2), generator=g, device=DEVICE, dtype=torch.int32).to(torch.uint8)
        if C % 2:
            codes[:, -1] &= 15
        state["codes"] = codes
        return state
    state["A"] = _matrix(case, g)
    state["dims"], state["thresholds"] = _trees(case, state["A"], seed)
    state["params"] = m.Params(state["dims"], state["thresholds"])
    return state


def run(state):
    case = state["case"]
    call = case["call"]
    if call == "learn":
        p = m.learn_on_device(state["A"], state["subspaces"])
        return [p.split_dims, p.thresholds, p.prototypes]
    if call == "tables":
        return list(m.maddness_build_luts(state["params"], state["B"]))
    if call == "scan":
        return m.maddness_scan(case["C"], state["codes"], state["luts"], state["scale"], state["offset"])[0]
    plain = case["dtype"] == "f32" and not case["columns"]
    if call == "encode":
        if plain:
            return m.maddness_encode(state["params"], state["A"])
        return m.maddness_encode_typed(state["params"], state["A"], col_major=case["columns"])
    tables = (state["luts"], state["scale"], state["offset"])
    if call == "averaged":
        return m.maddness_encode_scan_averaged(state["params"], state["A"], *tables)
    if plain:
        return m.maddness_encode_scan(state["params"], state["A"], *tables)
    return m.maddness_encode_scan_typed(state["params"], state["A"], *tables, col_major=case["columns"])


def work(case):
    call, N, D, M, C = (case[k] for k in ("call", "N", "D", "M", "C"))
    size = DTYPES[case["dtype"]].itemsize
    tree, luts, packed = C * 80, C * 16 * M + 8 * M, (C + 1) // 2
    read = N * size * (min(D, 4 * C) if case["columns"] else D)
    if call == "learn":
        Q = 16 * C
        # four levels of a sort and the two running sums over each candidate, then the ridge system: G^T A, its
        # factor and two triangular solves for D right-hand sides
        sums = 4 * min(4, D // C) * N * (6 * D + C * math.log2(max(N, 2)))
        return {"bytes": 4 * N * D + C * 80 + 4 * Q * D, "flops": sums + N * C * D + Q ** 3 / 3 + 2 * Q * Q * D}
    if call == "tables":
        return {"bytes": 4 * (16 * C * D + D * M) + luts, "flops": 2 * 16 * C * D * M}
    if call == "scan":
        return {"bytes": N * packed + luts + 4 * N * M, "flops": N * M * C}
    if call == "encode":
        return {"bytes": read + tree + N * packed, "flops": 4 * N * C}
    return {"bytes": read + tree + luts + 4 * N * M, "flops": 4 * N * C + N * M * C}


def tolerance(case):
    if case["call"] == "tables":
        # 64-bit sums, in any order, rounded to fp32 (offset) or to a byte (an entry on the edge between two)
        return {"rel": 2.5e-7, "max": 5e-7, "differ": 1e-6}
    if case["call"] == "learn":
        # trees are whole numbers and midpoints of two values of the data; prototypes are 64-bit solutions
        # rounded to fp32
        return {"rel": 2.5e-7, "max": 1e-6}
    # the sum of bytes is exact, the scale a power of two: one rounding, the same in every correct implementation
    return "exact"


# ---------------------------------------------------------------------------------------------------------
# the same outputs from plain torch in 64 bits

def _codes(case, state, lo, n):
    """[n][C] codes of rows lo .. lo + n."""
    A = state["A"]
    X = (A[:, lo:lo + n].t() if case["columns"] else A[lo:lo + n]).double()
    th = state["thresholds"].double()
    at = torch.arange(case["C"], device=DEVICE)
    node = torch.zeros((n, case["C"]), dtype=torch.int64, device=DEVICE)
    for t in range(4):
        node = 2 * node + (X[:, state["dims"][:, t].long()] >= th[at, (1 << t) - 1 + node]).long()
    return node


def _pack(codes):
    if codes.shape[1] % 2:
        codes = torch.cat([codes, torch.zeros_like(codes[:, :1])], 1)
    return (codes[:, 0::2] | (codes[:, 1::2] << 4)).to(torch.uint8)


def _sums(case, luts, codes):
    """The aggregate of the looked-up entries, in whole numbers."""
    if case["call"] == "averaged":
        total = 0
        for block in range(0, case["C"], 16):
            level = [luts[c][codes[:, c]].int() for c in range(block, block + 16)]
            while len(level) > 1:
                level = [(a + b + 1) >> 1 for a, b in zip(level[0::2], level[1::2])]
            total = total + level[0]
        return 16 * total - case["C"]
    acc = torch.zeros((codes.shape[0], luts.shape[2]), dtype=torch.int32, device=DEVICE)
    for c in range(case["C"]):
        acc += luts[c][codes[:, c]]
    return acc


def _grow(A, subspaces):
    """Algorithms 2-4 of the paper on one training matrix: (split columns, thresholds, codes), sums in 64 bits."""
    N = A.shape[0]
    dims = torch.zeros((len(subspaces), 4), dtype=torch.int32)
    thresholds = torch.zeros((len(subspaces), 16))
    codes = torch.zeros((N, len(subspaces)), dtype=torch.int64, device=DEVICE)
    for c, (lo, hi) in enumerate(subspaces):
        X, X32 = A[:, lo:hi].double(), A[:, lo:hi]
        node = torch.zeros(N, dtype=torch.int64, device=DEVICE)
        for t in range(4):
            rows = [torch.nonzero(node == b).flatten() for b in range(1 << t)]
            spread = sum((X[r] - X[r].mean(0)).square().sum(0) if len(r) else X.new_zeros(hi - lo) for r in rows)
            best = None
            for j in torch.argsort(spread, descending=True, stable=True)[:4].tolist():
                loss, cut = 0.0, []
                for r in rows:
                    x = X32[r, j]
                    if len(r) < 2 or bool(x.min() == x.max()):
                        loss += float((X[r] - X[r].mean(0)).square().sum()) if len(r) else 0.0
                        cut.append(float(x[0]) if len(r) else 0.0)
                        continue
                    x, order = torch.sort(x, stable=True)
                    Y = X[r][order]
                    n = torch.arange(1, len(r) + 1, device=DEVICE, dtype=torch.float64)[:, None]
                    head = (Y.square().cumsum(0) - Y.cumsum(0).square() / n).sum(1)
                    Z = Y.flip(0)
                    tail = (Z.square().cumsum(0) - Z.cumsum(0).square() / n).sum(1).flip(0)
                    both = torch.where(x[:-1] < x[1:], head[:-1] + tail[1:], torch.inf)
                    at = int(torch.argmin(both))
                    a, b = x[at].cpu(), x[at + 1].cpu()
                    v = ((a.double() + b.double()) / 2).float()
                    loss += float(both[at])
                    cut.append(float(b if v <= a else v))
                if best is None or loss < best[0]:
                    best = (loss, j, cut)
            _, j, cut = best
            dims[c, t] = lo + j
            v = torch.tensor(cut)
            thresholds[c, (1 << t) - 1:(2 << t) - 1] = v
            node = 2 * node + (X32[:, j] >= v.to(DEVICE)[node]).long()
        codes[:, c] = node
    return dims.to(DEVICE), thresholds.to(DEVICE).double(), codes


def exact(case, seed):
    state = prepare(case, seed)
    call, N, D, M, C = (case[k] for k in ("call", "N", "D", "M", "C"))
    if call == "learn":
        dims, thresholds, codes = _grow(state["A"], state["subspaces"])
        G = torch.zeros((N, 16 * C), dtype=torch.float64, device=DEVICE)
        G.scatter_(1, codes + 16 * torch.arange(C, device=DEVICE), 1.0)
        H = G.t() @ G + torch.eye(16 * C, dtype=torch.float64, device=DEVICE)
        P = torch.cholesky_solve(G.t() @ state["A"].double(), torch.linalg.cholesky(H))
        return [dims, thresholds, P.reshape(C, 16, D)]
    if call == "tables":
        T = (state["params"].prototypes.double().reshape(16 * C, D) @ state["B"].double()).reshape(C, 16, M)
        delta = T.amin(1, keepdim=True)
        widest = (T - delta).amax((0, 1))
        power = torch.floor(torch.log2(255 / widest))
        power = torch.where(widest * torch.exp2(power + 1) <= 255, power + 1, power)
        power = torch.where(widest * torch.exp2(power) > 255, power - 1, power).clamp(-126, 126)
        luts = ((T - delta) * torch.exp2(power)).round().clamp(0, 255).to(torch.uint8)
        return [luts, torch.exp2(-power), delta.sum((0, 1))]
    if call == "encode":
        return torch.cat([_pack(_codes(case, state, lo, min(PIECE, N - lo))) for lo in range(0, N, PIECE)])
    luts, scale, offset = state["luts"], state["scale"].double(), state["offset"].double()
    out = torch.empty((N, M), dtype=torch.float64, device=DEVICE)
    for lo in range(0, N, PIECE):
        n = min(PIECE, N - lo)
        if call == "scan":
            packed = state["codes"][lo:lo + n].long()
            codes = torch.stack([packed & 15, packed >> 4], 2).reshape(n, -1)[:, :C]
        else:
            codes = _codes(case, state, lo, n)
        out[lo:lo + n] = _sums(case, luts, codes) * scale + offset
    return out

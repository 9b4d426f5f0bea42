"""How far the learner's estimates may be off (csrc/learn_bounds.h) against what they and the sums in the algorithms' order
really are off, by whole numbers of any size."""
import ctypes
import os
import subprocess
from fractions import Fraction

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2106_10860_amd", "csrc")


@pytest.fixture(scope="module")
def bounds(tmp_path_factory):
    folder = tmp_path_factory.mktemp("bounds")
    (folder / "b.cpp").write_text(
        '#include "learn_bounds.h"\n'
        'extern "C" double loss(double n, double sy, double p) { return maddness::loss_error(n, sy, p); }\n'
        'extern "C" double split(double n, double root, double rows, double energy, int d, int exact, int every)\n'
        '{ return maddness::split_error(n, root, rows, energy, d, exact, every); }\n')
    out = str(folder / "b.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-shared", "-fPIC", "-I", CSRC, str(folder / "b.cpp"), "-o", out])
    L = ctypes.CDLL(out)
    L.loss.restype = L.split.restype = ctypes.c_double
    L.loss.argtypes = [ctypes.c_double] * 3
    L.split.argtypes = [ctypes.c_double] * 4 + [ctypes.c_int] * 3
    return L


def chain(x):
    """The sum in order (numpy's running sums are)."""
    return float(np.cumsum(x)[-1])


def two_passes(x):
    """L(j, B) as the exact kernel has it."""
    return chain((x - chain(x) / len(x)) ** 2)


@pytest.mark.parametrize("log2n", [10, 18, 20, 22])
@pytest.mark.parametrize("share", [0.5, 0.3, 0.1])
def test_loss_of_a_bucket_that_is_not_split(bounds, log2n, share):
    """Binary values: every sum of them is exact, the squared distances from their mean are not, and round the same way term after
    term.  The bounds cover it, for the choice of columns and for that among candidates where one cannot split the bucket."""
    n = (1 << log2n) - 1
    ones = int(n * share) | 1
    x = np.zeros(n)
    x[np.random.default_rng(1).permutation(n)[:ones]] = 1.0
    off = abs(Fraction(two_passes(x)) - Fraction(ones * (n - ones), n))
    assert off <= bounds.split(n, n ** 0.5, n, ones, 1, 1, 0)
    assert off <= bounds.loss(n, ones, 0.0) and off <= bounds.loss(n, n - ones, 1.0)


def whole(x):
    """fp32 values as whole numbers times 2^-e."""
    e = 149
    return np.array([int(Fraction(float(v)) * (1 << e)) for v in x], dtype=object), e


@pytest.mark.parametrize("kind", ["normal", "far", "whole", "few", "wide"])
@pytest.mark.parametrize("n", [2, 33, 3000])
def test_estimates_and_chains_stay_within_the_bounds(bounds, kind, n):
    rng = np.random.default_rng(n)
    d = 3
    x = {"normal": lambda: rng.standard_normal((n, d)), "far": lambda: 1000 + 1e-3 * rng.standard_normal((n, d)),
         "whole": lambda: rng.integers(0, 256, (n, d)), "few": lambda: rng.integers(0, 2, (n, d)),
         "wide": lambda: rng.standard_normal((n, d)) * 10.0 ** rng.integers(-6, 6, (n, d))}[kind]().astype(np.float32).astype(np.float64)
    exact_sums = kind in ("whole", "few")
    w, e = zip(*(whole(x[:, j]) for j in range(d)))
    one = Fraction(1, 1 << e[0])
    T, Q = [sum(v) * one for v in w], [sum(v * v) * one * one for v in w]
    energy = float(sum(Q))
    for j in range(d):
        p = x[n // 2, j]
        y = x[:, j] - p
        true, pivoted = Q[j] - T[j] * T[j] / n, np.sum(y * y) - np.sum(y) ** 2 / n
        assert abs(Fraction(two_passes(x[:, j])) - true) + abs(Fraction(float(max(pivoted, 0.0))) - true) <= bounds.loss(n, float(np.sum(y * y)), p)
    # a split after row r: the chains up and down, and a constant less the gain
    up, up2 = np.cumsum(x, 0), np.cumsum(x * x, 0)
    down, down2 = np.cumsum(x[::-1], 0)[::-1], np.cumsum(x[::-1] ** 2, 0)[::-1]
    for r in sorted({0, n // 3, n // 2, n - 2}):
        n1 = r + 1
        loss = sum(up2[r, j] - up[r, j] ** 2 / n1 + down2[n1, j] - down[n1, j] ** 2 / (n - n1) for j in range(d)) if n1 < n else None
        if loss is None:
            continue
        heads = [sum(w[j][:n1]) * one for j in range(d)]
        gain = sum((heads[j] - T[j] * n1 / n) ** 2 * n / (n1 * (n - n1)) for j in range(d))
        true = sum(Q[j] - T[j] * T[j] / n for j in range(d)) - gain
        s = [np.sum(x[:n1, j]) for j in range(d)]
        estimate = sum((s[j] - n1 * (np.sum(x[:, j]) / n)) ** 2 for j in range(d)) * n / (n1 * (n - n1))
        off = abs(Fraction(float(loss)) - true) + abs(Fraction(float(estimate)) - gain)
        assert off <= bounds.split(n, n ** 0.5, n, energy, d, exact_sums, 1)

"""The native argument marshalling: the calls it takes give what the Python marshalling gives, and what it does not take
(other types, shapes, tensors that are not plain) is accepted or refused as it was."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mad():
    import torch
    import paper_2106_10860_amd as m
    assert torch.cuda.is_available()
    m.lib()
    return m


class Watched:
    """The native marshalling; `taken` says of each call whether it did it (a status is one it did) or left it to the Python code."""

    def __init__(self, native):
        self.native, self.taken = native, []

    def __getattr__(self, name):
        def call(*args):
            r = getattr(self.native, name)(*args)
            self.taken.append(r is not NotImplemented)
            return r
        return call


@pytest.fixture
def both(mad, monkeypatch):
    """f -> (result through the native marshalling, result without it, whether the native one did it)"""
    def run(f):
        def outcome():
            try:
                return f()
            except Exception as e:
                return type(e), str(e)
        with monkeypatch.context() as mp:
            watched = Watched(mad._native)
            mp.setattr(mad, "_native", watched)
            native = outcome()
            mp.setattr(mad, "_native", mad._NotBuilt)
            return native, outcome(), all(watched.taken) and len(watched.taken) == 1
    return run


def same(x, y):
    import torch
    if isinstance(x, (tuple, list)):
        return len(x) == len(y) and all(same(a, b) for a, b in zip(x, y))
    if isinstance(x, torch.Tensor):
        return isinstance(y, torch.Tensor) and x.dtype == y.dtype and x.shape == y.shape and x.stride() == y.stride() and torch.equal(x, y)
    return x == y


def test_native_marshalling(mad, both):
    import torch
    g = torch.Generator(device="cuda").manual_seed(3)
    N, D, M, C = 100, 64, 24, 8
    A = torch.randn((N, D), device="cuda", generator=g)
    P = torch.randn((C, 16, D), device="cuda", generator=g)
    trees = (torch.randint(0, D, (C, 4), dtype=torch.int32, device="cuda", generator=g), torch.randn((C, 16), device="cuda", generator=g))
    params, dense = mad.Params(*trees), mad.Params(*trees, P)
    B = torch.randn((D, M), device="cuda", generator=g)
    luts, scale, offset = mad.maddness_build_luts(dense, B)
    assert mad._native.__name__ == "maddness_binding"
    tables = (luts, scale, offset)
    codes = mad.maddness_encode(params, A)
    wide = torch.zeros((N, M + 3), device="cuda")
    side = torch.cuda.Stream()

    def on_side():
        side.wait_stream(torch.cuda.current_stream())
        out = mad.maddness_encode_scan(params, A, *tables, stream=side)
        torch.cuda.current_stream().wait_stream(side)
        return out

    acc = torch.zeros((N, M), dtype=torch.int16, device="cuda")
    wide_acc = torch.zeros((N, M), dtype=torch.int16, device="cuda").view(torch.uint16)
    half, by_columns = A.half(), A.half().t().contiguous()

    class Plain(torch.Tensor):
        pass

    C2 = 16
    trees2 = (torch.randint(0, D, (C2, 4), dtype=torch.int32, device="cuda", generator=g), torch.randn((C2, 16), device="cuda", generator=g))
    params2, tables2 = mad.Params(*trees2), (torch.randint(0, 256, (C2, 16, M), dtype=torch.uint8, device="cuda", generator=g), scale, offset)
    codes2, kept = mad.maddness_encode(params2, A), torch.zeros_like(codes)
    taken = [
        lambda: mad.maddness_encode(params, A), lambda: mad.maddness_encode_typed(params, by_columns, col_major=True),
        lambda: mad.maddness_encode_scan(params, A, *tables), lambda: mad.maddness_encode_scan(params, A, *tables, out=wide[:, :M]),
        lambda: (mad.maddness_encode_scan(params, A, *tables, acc=acc, want_out=False), acc.clone()),
        lambda: (mad.maddness_encode_scan(params, A, *tables, acc=wide_acc, codes=kept), wide_acc.view(torch.int16).clone(), kept.clone()),
        lambda: mad.maddness_encode_scan_typed(params, half, *tables), lambda: mad.maddness_encode_scan(params, A[:0], *tables),
        lambda: mad.maddness_encode_scan_typed(params, by_columns, *tables, col_major=True),
        lambda: mad.maddness_encode_scan_averaged(params2, A, *tables2),
        lambda: mad.maddness_scan(C, codes, *tables), lambda: mad.maddness_scan_averaged(C2, codes2, *tables2),
        lambda: mad.maddness_scan(C, codes, *tables, out=wide[:, :M], acc=acc),
        lambda: mad.maddness_scan(C, codes, *tables, acc=acc, want_out=False),
        lambda: mad.maddness_build_luts(dense, B), on_side, lambda: mad.maddness_encode_scan(params, torch.nn.Parameter(A), *tables),
        lambda: mad.maddness_build_luts_pooled(dense, B), lambda: mad.maddness_encode_scan(params, A[5:6], *tables),
        # refused by the library
        lambda: mad.maddness_encode_scan_averaged(params, A, *tables), lambda: mad.maddness_scan(0, codes, *tables),
        lambda: mad.maddness_build_luts(dense, B, workspace=torch.empty(4, dtype=torch.uint8, device="cuda")),
    ]
    left = [
        lambda: mad.maddness_encode_scan(params, A.as_subclass(Plain), *tables),
        # refused before the library
        lambda: mad.maddness_encode(params, A.cpu()), lambda: mad.maddness_encode(params, A.double()),
        lambda: mad.maddness_encode(params, A.t()), lambda: mad.maddness_encode(params, A[0]), lambda: mad.maddness_encode(params, None),
        lambda: mad.maddness_encode(dense, A[:, :8].contiguous()), lambda: mad.maddness_encode_scan(params, half, *tables),
        lambda: mad.maddness_encode_scan(params, A, luts.int(), scale, offset),
        lambda: mad.maddness_encode_scan(params, A, luts, scale.double(), offset), lambda: mad.maddness_build_luts(params, B),
        lambda: mad.maddness_encode_scan(params, A, *tables, out=torch.empty((M, N), device="cuda").t()),
        lambda: mad.maddness_encode_scan_typed(params, A.int(), *tables),
    ]
    either = [lambda: mad.maddness_encode_scan(params, A, luts, None, offset)]     # (a null pointer, which the library refuses)
    for k, call in enumerate(taken + left + either):
        x, y, native = both(call)
        torch.cuda.synchronize()
        assert same(x, y), (k, x, y)
        assert k >= len(taken) + len(left) or native == (k < len(taken)), (k, native, x)
    given = torch.empty((N, M), device="cuda")
    assert mad.maddness_encode_scan(params, A, *tables, out=given) is given
    assert mad.maddness_encode(params, A, codes=codes) is codes

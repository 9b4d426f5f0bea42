"""A native marshalling that is missing, broken or built for another torch: the calls go on without it, and a warning says so."""
import os
import shutil
import warnings

import pytest


@pytest.fixture
def mad(monkeypatch):
    pytest.importorskip("torch")
    import paper_2106_10860_amd as m
    if not (os.path.exists(m.LIB_PATH) and os.path.exists(m.NATIVE_PATH)):
        pytest.skip("not built")
    m.lib()
    monkeypatch.setattr(m, "_native", m._NotLoaded())
    return m


def encode_host_tensor(m):
    """A call that the Python marshalling refuses with a message of its own."""
    import torch
    params = m.Params(torch.zeros((2, 4), dtype=torch.int32), torch.zeros((2, 16)))
    with pytest.raises(TypeError, match="A must be a device tensor|split_dims must be a device tensor"):
        m.maddness_encode(params, torch.zeros((3, 5)))


@pytest.mark.parametrize("kind", ["missing", "broken", "other_torch"])
def test_calls_without_a_native_marshalling_that_loads(mad, monkeypatch, tmp_path, kind):
    import torch
    path = tmp_path / "maddness_binding.so"
    if kind == "broken":
        path.write_bytes(b"no library")
    elif kind == "other_torch":
        shutil.copy(mad.NATIVE_PATH, path)
        os.symlink(mad.LIB_PATH, tmp_path / "libmaddness.so")
        monkeypatch.setattr(torch, "__version__", "0.0.0")
    monkeypatch.setattr(mad, "NATIVE_PATH", str(path))
    with pytest.warns(RuntimeWarning, match="native argument marshalling" if kind != "other_torch" else "this is torch 0.0.0"):
        encode_host_tensor(mad)
    assert mad._native is mad._NotBuilt
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        encode_host_tensor(mad)         # (said once)


def test_native_marshalling_loads_as_built(mad, tmp_path, monkeypatch):
    shutil.copy(mad.NATIVE_PATH, tmp_path / "maddness_binding.so")
    os.symlink(mad.LIB_PATH, tmp_path / "libmaddness.so")
    monkeypatch.setattr(mad, "NATIVE_PATH", str(tmp_path / "maddness_binding.so"))
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        encode_host_tensor(mad)
    assert mad._native.__name__ == "maddness_binding"


def test_library_is_built_where_torch_is_not(monkeypatch, tmp_path, capsys):
    from paper_2106_10860_amd import build
    stale = tmp_path / "maddness_binding.so"
    stale.write_bytes(b"")
    monkeypatch.setattr(build, "BINDING_LIB", str(stale))
    monkeypatch.setenv("CXX", str(tmp_path / "no_compiler"))
    assert build.build_binding() is False
    assert not stale.exists() and "is not built" in capsys.readouterr().err

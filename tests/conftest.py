import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


def _has_gpu() -> bool:
    try:
        import torch
        return torch.cuda.is_available()
    except Exception:
        return False


def pytest_collection_modifyitems(config, items):
    if _has_gpu():
        return
    skip = pytest.mark.skip(reason="no GPU visible")
    for item in items:
        if "gpu" in item.keywords:
            item.add_marker(skip)


@pytest.fixture(params=[True, False], ids=["auto", "no_blocks"])
def blocks(request):
    """Every shape twice: with the library's own choice of kernels, and without the one that works by blocks of rows and columns, so
    that the kernels beside it are reached with the shapes that it would take."""
    import paper_2106_10860_amd as m
    if not request.param:
        m.maddness_set_option(m.MADDNESS_OPT_MAX_WORKGROUPS, 1 << 20)       # (more than any of them launches)
    yield request.param
    m.maddness_set_option(m.MADDNESS_OPT_MAX_WORKGROUPS, 0)

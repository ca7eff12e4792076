import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(params=["spans", "128", "256"])
def cut(request, monkeypatch):
    """The three ways to cut a launch, whichever is chosen at its size: queries of its units, 0 in spans."""
    monkeypatch.setenv("DF_ATTN_CUT", request.param)
    return 0 if request.param == "spans" else int(request.param)


def pytest_collection_modifyitems(config, items):
    # GPU tests are skipped, not failed, when no device is present and -m gpu was not asked for.
    try:
        import torch
        has_gpu = torch.cuda.is_available()
    except Exception:  # pragma: no cover
        has_gpu = False
    if has_gpu:
        return
    skip = pytest.mark.skip(reason="no GPU in this environment")
    for item in items:
        if "gpu" in item.keywords:
            item.add_marker(skip)
